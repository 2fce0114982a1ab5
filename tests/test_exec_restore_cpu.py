"""Code-generation guard (CPU only): no register copy before the lanes are back.

At the end of a divergent loop or branch the join block first restores the
EXEC mask (``s_or_b64 exec, exec, ...``).  This compiler can place copies that
it makes of vector registers living across a call (or reloads and spills of
them) at the top of that block, in front of the restore, when scalar registers
are saved to vector lanes there: the copies then run without the lanes that
left the loop -- after a loop, without any lane -- and those lanes go on with
garbage.  A build that had this in front of the call of the gather sort, with
the registers of the cross-lane sums, returned wrong counts and did not end.
"""
import os
import re
import subprocess
import sys
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_0912_2555_amd", "csrc", "mapcheck.hip")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

RESTORE = re.compile(r"s_or_b64 exec, exec, s\[")
WHOLE_WAVE = re.compile(r"s_or_saveexec_b64 s\[\d+:\d+\], -1|s_mov_b64 exec, -1")
COPY = re.compile(r"v_mov_b(32_e32|64_e32) v\S+, v|v_accvgpr_\S+ |scratch_(load|store)\S* .*Folded")
QUIET = re.compile(r"s_|v_(readlane|writelane|mov_b|accvgpr)|scratch_")


def early_copies(asm):
    """(function, block, instruction) of every vector register copy, spill or reload that precedes, in its basic
    block, the EXEC restore the block begins with (only scalar instructions, lane moves and other copies before)."""
    found, func, block, before, whole = [], None, None, [], False
    for line in asm.split("\n"):
        t = line.strip()
        m = re.match(r"^([A-Za-z_][\w.$]*):", line)
        if m and not t.startswith(".L"):
            func = m.group(1)
        if t.startswith((".LBB", "; %bb.")) or (m and not t.startswith(".L")):
            block, before, whole = t.split()[0], [], False
            continue
        if not t or t.startswith((";", ".")) or before is None:
            continue
        if WHOLE_WAVE.match(t):
            whole = True
        elif re.match(r"s_mov_b64 exec, s\[", t):
            whole = False
        elif RESTORE.match(t):
            found += [(func, block, x) for x in before]
            before = None
        elif not QUIET.match(t):
            before = None
        elif COPY.match(t) and not whole:
            before.append(t)
    return found


def test_scanner_sees_a_copy_before_the_restore():
    bad = ("f:\n.LBB0_1:\n\tv_writelane_b32 v126, s36, 14\n\tv_mov_b32_e32 v90, v53\n\ts_nop 0\n"
           "\ts_or_b64 exec, exec, s[16:17]\n\ts_swappc_b64 s[30:31], s[0:1]\n")
    assert early_copies(bad) == [("f", ".LBB0_1:", "v_mov_b32_e32 v90, v53")]
    assert early_copies(bad.replace("v90, v53", "v90, 0")) == []
    assert early_copies(bad.replace("\tv_mov_b32_e32 v90, v53\n", "").replace(
        "\ts_swappc", "\tv_mov_b32_e32 v90, v53\n\ts_swappc")) == []
    assert early_copies("f:\n.LBB0_1:\n\ts_or_saveexec_b64 s[0:1], -1\n\tscratch_load_dword v58, off, s32 ; 4-byte "
                        "Folded Reload\n\ts_mov_b64 exec, s[0:1]\n\ts_or_b64 exec, exec, s[4:5]\n") == []


def test_no_register_copy_precedes_an_exec_restore():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    sys.path.insert(0, os.path.join(ROOT, "paper_0912_2555_amd"))
    try:
        import build as hipbuild
    finally:
        sys.path.pop(0)
    flags = [f for f in hipbuild.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "mapcheck.s")
        subprocess.check_call([HIPCC, *flags, "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-S", "-o",
                               out, SRC], stderr=subprocess.DEVNULL)
        assert early_copies(open(out).read()) == []
