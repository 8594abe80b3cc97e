"""The deal of the attention kernel's work to wavefronts (units of fp rows, tiles of quantized rows): the kernel's own
arithmetic, csrc/lq_schedule.h, compiled for the host and run for random launches of all four programs, the tiles
that are drawn at run time in a random order.  A unit or tile that is left out would silently drop tokens."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2503_19950_amd", "csrc")


def test_every_unit_and_tile_is_taken_once(tmp_path):
    exe = tmp_path / "schedule"
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe),
                    os.path.join(HERE, "host", "schedule.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
