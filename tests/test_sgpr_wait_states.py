"""The built kernels' assembly, read from libmialign.so: on gfx950 a VALU instruction that reads an SGPR (a lane mask, say)
must come at least two wait states after the VALU instruction that wrote it.  The compiler keeps them for its own
instructions, not for an instruction inside inline asm, so every one is checked here, in the order of the code."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2002_04561_amd as aln

LIB = os.path.join(os.path.dirname(os.path.abspath(aln.__file__)), "libmialign.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 2
VCC = (106, 107)
# a second destination (a carry or a flag) follows the first
TWO_DST = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[iu]64_")


def sgprs(arg):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", arg)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", arg)
    if m:
        return {int(m[1])}
    return {"vcc": set(VCC), "vcc_lo": {VCC[0]}, "vcc_hi": {VCC[1]}}.get(arg, set())


def early_reads(text):
    """(VALU instructions that read SGPRs, those of them that come too early) in a disassembly."""
    reads, early = 0, []
    written = []  # (wait states since, registers)
    where = ""
    for line in text.split("\n"):
        m = re.match(r"(?:[0-9a-f]+ )?<(\S+)>:", line)
        if m:
            where, written = m[1], []
            continue
        line = line.split("//")[0].strip()
        if not line:
            continue
        op, _, rest = line.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        n_dst = 2 if TWO_DST.match(op) else 1
        valu = op.startswith("v_")
        if valu:
            src = set().union(*[sgprs(a) for a in args[n_dst:]]) if len(args) > n_dst else set()
            reads += bool(src)
            early += [(where, line) for age, regs in written if age < WAIT_STATES and regs & src]
        states = int(args[0], 0) + 1 if op == "s_nop" else 1
        written = [(age + states, regs) for age, regs in written if age + states < WAIT_STATES]
        if valu:
            dst = set().union(*[sgprs(a) for a in args[:n_dst]])
            if dst:
                written.append((0, dst))
        elif op in ("s_branch", "s_endpgm"):
            written = []
    return reads, early


def test_scan_finds_a_short_distance():
    ok = "<k>:\n v_cmp_eq_u32_e64 s[4:5], v0, v1\n s_nop 1\n v_cndmask_b32_e64 v2, v3, v4, s[4:5]\n"
    assert early_reads(ok) == (1, [])
    assert len(early_reads(ok.replace("s_nop 1", "s_nop 0"))[1]) == 1
    assert len(early_reads(ok.replace("s_nop 1", "v_mov_b32_e32 v9, v8"))[1]) == 1
    assert early_reads(ok.replace("s_nop 1", "v_mad_u64_u32 v[8:9], s[4:5], v6, v7, 0\n s_nop 1")) == (1, [])
    assert len(early_reads("<k>:\n v_cmp_eq_u32_e32 vcc, v0, v1\n v_cndmask_b32_e32 v2, v3, v4, vcc\n")[1]) == 1


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_masks_are_read_two_wait_states_after_they_are_written(tmp_path):
    assert os.path.exists(LIB), "library not built"
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    objs = sorted(p for p in os.listdir(tmp_path) if "gfx950" in p)
    assert objs
    reads, early = 0, []
    for p in objs:
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", p], cwd=tmp_path, check=True,
                           capture_output=True, text=True)
        n, e = early_reads(r.stdout)
        reads += n
        early += e
    assert reads > 10000, reads  # the kernels were disassembled
    assert not early, (len(early), early[:3])
