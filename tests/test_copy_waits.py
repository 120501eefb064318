"""Wait states of the global-to-LDS copies. They are inline assembly, which the
compiler's hazard recognizer does not look into, so the assembly it generates
around them is checked here: a copy reads M0 (its LDS address) at least one wait
state after a scalar write of M0, and its scalar base at least five wait states
after a vector instruction (v_readlane, v_readfirstlane, a compare) wrote it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2608_19758_amd import build

# wait states between a write of the operand and the copy that reads it
M0_STATES, BASE_STATES = 1, 5


def _instructions(text):
    """(mnemonic, operand text) of every instruction, None at a label."""
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"^[\w.$]+:$", line):
            yield None
        elif line and not line.startswith((".", "//")):
            yield tuple(line.split(None, 1)) if " " in line or "\t" in line else (line, "")


def _sregs(text):
    """Scalar registers named in an operand."""
    regs = set()
    for a, b, c in re.findall(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        regs |= {int(c)} if c else set(range(int(a), int(b) + 1))
    return regs


def hazards(text):
    """(copies, list of copies that read an operand too early)."""
    ins = list(_instructions(text))
    copies, bad = 0, []
    for at, cur in enumerate(ins):
        if cur is None or not cur[0].startswith("global_load_lds"):
            continue
        copies += 1
        base = _sregs(cur[1].split(",", 1)[1])
        states, k, need = 0, at - 1, BASE_STATES if base else M0_STATES
        while states < need and k >= 0:
            if ins[k] is None:   # another path may come in here: nothing is known of it
                bad.append((at, "label", cur))
                break
            op, args = ins[k]
            if op == "s_nop":
                states += int(args, 0) + 1
            else:
                dst = args.split(",")[0]
                if op.startswith("s_") and dst == "m0" and states < M0_STATES:
                    bad.append((at, op, cur))
                if op.startswith("v_") and base & _sregs(dst):
                    bad.append((at, op, cur))
                states += 1
            k -= 1
    return copies, bad


def test_checker():
    ok = "s_mov_b32 m0, s4\ns_nop 3\nglobal_load_lds_dwordx4 v1, s[6:7]\n"
    assert hazards("v_readlane_b32 s6, v9, 1\n" + ok) == (1, [])
    early = ok.replace("s_nop 3", "s_nop 2")
    assert len(hazards("v_readlane_b32 s7, v9, 1\n" + early)[1]) == 1
    assert len(hazards(early.replace("s_nop 2\n", ""))[1]) == 1
    assert hazards("s_add_u32 s6, s6, s8\ns_mov_b32 s9, 0\ns_mov_b32 s9, 0\n" + early) == (1, [])


@pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)), reason="no hipcc")
def test_copies_wait_for_their_operands(tmp_path):
    out = tmp_path / "attend.s"
    subprocess.run([build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", "-o", str(out),
                                                  os.path.join(build.CSRC, "attend.hip")],
                   check=True, capture_output=True)
    copies, bad = hazards(out.read_text())
    print("%d copies" % copies)
    assert copies > 0
    assert not bad, bad[:4]
