"""The quantizers' quotient by the block's reciprocal (`recip_quotient.h`)
equals the IEEE quotient for every bf16 input: plain C++, compiled here with
g++, so this runs without a GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_27875_amd", "csrc")


def test_every_quotient_is_correctly_rounded(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "recip_check")
    # no contraction: every step is the one the header writes
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(HERE, "recip_check.cpp"), "-o", exe], check=True)
    pairs, bad = map(int, subprocess.run([exe], capture_output=True, text=True).stdout.split())
    assert pairs > 10_000_000 and bad == 0, (pairs, bad)
