"""Host test of the work queue's claims with emulated lanes (no device): compiles
tests/queue_claim_test.cpp with g++ against the queue's header and runs it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_claims_agree_in_all_lanes(tmp_path):
    exe = str(tmp_path / "queue_claim_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread",
                    "-I" + os.path.join(ROOT, "paper_1309_2710_amd", "csrc"),
                    os.path.join(ROOT, "tests", "queue_claim_test.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout
