"""Waits that neither the hardware nor the compiler inserts around hand-written
instructions, checked in the generated gfx950 assembly of every kernel that
has them (no GPU).  A direct global -> LDS copy must not follow the write of M0
(its LDS address) at once, and its scalar base must not have been written by a
vector instruction within the five wait states before it."""

import os
import re
import subprocess

import pytest

from paper_2608_07524_amd import build as B

COPY = re.compile(r"global_load_lds_dword(x4)? ")


def _assembly(source, out):
    cmd = [B._hipcc(), "-x", "hip", *B.COMMON_FLAGS, "--cuda-device-only", "-S", *B.DEVICE_FLAGS, source, "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    lines = [l.split(";")[0].strip() for l in open(out)]
    return [l for l in lines if l and (l.endswith(":") or not l.startswith("."))]


def _regs(operand):
    m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    lo = int(m[1] or m[2])
    return set(range(lo, int(m[3] or lo) + 1))


def _violations(code):
    """Copies reached, along some path, too soon after a write they read."""
    jumps = {}  # label -> instructions that branch to it
    for i, l in enumerate(code):
        m = re.match(r"s_c?branch\S* (\S+)", l)
        if m:
            jumps.setdefault(m[1] + ":", []).append(i)

    def writes_within(i, states, hit):
        """Whether a line matching ``hit`` lies less than ``states`` wait
        states before the instruction after line i."""
        while i >= 0 and states > 0:
            l = code[i]
            if l.endswith(":"):
                if any(writes_within(j, states, hit) for j in jumps.get(l, ())):
                    return True
                if i and re.match(r"s_(branch|endpgm)", code[i - 1]):
                    return False  # no fall-through
            elif hit(l):
                return True
            else:
                m = re.match(r"s_nop (\d+)", l)
                states -= int(m[1]) + 1 if m else 1
            i -= 1
        return False

    bad, n = [], 0
    for i, l in enumerate(code):
        if not COPY.match(l):
            continue
        n += 1
        base = _regs(l.split()[-1])
        vector_write = lambda x: x.startswith("v_") and bool(_regs(x.split()[1].rstrip(",")) & base)
        if writes_within(i - 1, 1, lambda x: re.match(r"s_\w+ m0,", x)) or writes_within(i - 1, 5, vector_write):
            bad.append(" / ".join(code[max(0, i - 6):i + 1]))
    return n, bad


def test_checker():
    m0 = ["s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3]"]
    assert _violations(m0)[1] and not _violations([m0[0], "s_nop 0", m0[1]])[1]
    vec = ["v_readfirstlane_b32 s3, v9", "s_mov_b32 m0, s4", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3]"]
    assert _violations(vec)[1] and not _violations(vec[:1] + ["s_nop 2"] + vec[1:])[1]
    assert not _violations(vec[:3] + ["global_load_lds_dwordx4 v1, s[4:5]"])[1]
    loop = ["s_nop 4", ".L:", "s_nop 0", "global_load_lds_dword v1, s[2:3]", "v_readlane_b32 s2, v0, 1", "s_cbranch_scc0 .L"]
    assert _violations(loop)[1] and not _violations(loop[:5] + ["s_nop 2"] + loop[5:])[1]


@pytest.mark.parametrize("name", ["attn_fwd.hip", "attn_bwd.hip", "layer_gemm.hip", "layer_proj.hip",
                                  "probe/dma_copy.hip"])
def test_waits_before_lds_copies(name, tmp_path):
    n, bad = _violations(_assembly(os.path.join(B.CSRC, name), str(tmp_path / "k.s")))
    assert n and not bad, (n, len(bad), bad[:3])


def test_every_source_with_copies_is_checked():
    found = []
    for base, _, files in os.walk(B.CSRC):
        for f in files:
            if re.search(r"lds_copy|load_lds|DmaTile<", open(os.path.join(base, f)).read()):
                found.append(f)
    assert sorted(found) == ["attn_bwd.hip", "attn_common.h", "attn_fwd.hip", "dma_copy.hip", "layer_gemm.hip",
                             "layer_proj.hip"]
