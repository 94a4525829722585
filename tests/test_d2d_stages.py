"""Device code of the registration's stage changes, one block at a time on
the CPU (tests/emulate): the shared state is read by all waves before a wave
that runs ahead writes it, whichever wave runs first, and every barrier is
reached by the whole block."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_state_between_stages_in_both_wave_orders(tmp_path):
    exe = str(tmp_path / "d2d_stages")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas",
                    "-I", os.path.join(ROOT, "tests", "emulate"),
                    "-I", os.path.join(ROOT, "paper_2307_00071_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "emulate", "d2d_stages.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "stages ok" in r.stdout
