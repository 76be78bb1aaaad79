"""CPU checks of the sample-domain channel mixing: its operand images against
the spherical harmonics and their orthonormality, and the rule that chooses
between it and the pair products at sizes that were measured both ways."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_10216_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_operand_images_and_rule(tmp_path):
    exe = str(tmp_path / "mixq_host")
    r = subprocess.run(["g++", "-O1", "-std=c++17", f"-I{CSRC}", "-o", exe,
                        os.path.join(ROOT, "tests", "mixq_host_main.cpp"), os.path.join(CSRC, "gtp_mixq_tables.cpp"),
                        os.path.join(CSRC, "gtp_tables.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout
