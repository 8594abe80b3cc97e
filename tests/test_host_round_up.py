"""The asm blocks that round towards +infinity (csrc/lq_round_up.h) write the mode register at both ends.  The hardware wants
two instructions (or an s_nop for them) between two such writes, which the compiler does not see to inside asm: also where
two blocks stand side by side.  Assembly only; nothing is run."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def waits_between_mode_writes(asm):
    """Instructions issued between each write of the mode register and the next one in the text, an s_nop N for N + 1; a
    label or a branch in between counts for nothing."""
    found, waits = [], None
    for line in asm.splitlines():
        words = re.sub(r"[;/].*", "", line).split()
        if not words or words[0].startswith(".") or words[0].endswith(":"):
            continue
        if words[0] == "s_endpgm":
            waits = None
        elif words[0].startswith("s_setreg"):
            assert "HW_REG_MODE" in line
            if waits is not None:
                found.append(waits)
            waits = 0
        elif waits is not None:
            waits += int(words[1]) + 1 if words[0] == "s_nop" else 1
    return found


def test_two_instructions_between_two_writes_of_the_mode(tmp_path):
    from paper_2503_19950_amd import build
    out = tmp_path / "device.s"
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.HIPCC_FLAGS, "-I", build.CSRC, "-S", "--cuda-device-only",
                        "-o", str(out), os.path.join(HERE, "host", "round_up_side_by_side.hip")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = waits_between_mode_writes(out.read_text())
    assert len(found) == 11 and min(found) >= 2, found
