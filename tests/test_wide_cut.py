"""The cut of wide token groups into pieces and the slots that the gate kernel hands to the down kernel (csrc/wide_cut.h), on the host:
every row slot and every h is read where it was written, no slot twice, for groups as the router leaves them, from evenly filled to all
tokens on one expert, in launches sized for the groups that were expected.  And the plans (csrc/wide_plan.h): no layer that the argument
checks accept has more segments than the down kernel's table."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_05950_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pieces_meet_where_they_were_put_and_fit_the_table(tmp_path):
    exe = str(tmp_path / "wide_cut")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-I", CSRC, os.path.join(HERE, "wide_cut_main.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert run.returncode == 0 and run.stdout.startswith("ok "), run.stdout[-2000:]
