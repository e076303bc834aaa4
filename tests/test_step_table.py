"""The packed entries in which a whole step's layers travel to its launches (csrc/st3_step.h), on the host: every field comes back,
and a layer whose values an entry cannot hold is refused (it takes a launch of its own)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_entries_hold_what_they_are_given(tmp_path):
    exe = str(tmp_path / "step_table")
    csrc = os.path.join(HERE, "..", "paper_2412_20105_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", csrc,
                    os.path.join(HERE, "step_table_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
