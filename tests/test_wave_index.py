"""Host test of the one-cell-per-wave kernels' index into the pressure-dependent
records (no device): compiles tests/wave_index_test.cpp with g++ against the
index's header and runs it; its forms are those that the library compiles."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_2710_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pressure_dependent_records_in_range(tmp_path):
    exe = str(tmp_path / "wave_index_test")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I" + CSRC,
                    os.path.join(ROOT, "tests", "wave_index_test.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout


def test_forms_of_the_library():
    """(lanes of the plan, unit rounds, waves per cell) of the pressure-dependent
    rows, as the host test has them."""
    rows = open(os.path.join(CSRC, "rkc_variants_wave.hip")).read()
    rows = rows[rows.index("kTable[] = {"):]
    have = {(int(a), int(c), int(d)) for a, c, d in re.findall(
        r"RKC_WAVE_PD\([\d.]+, \d+, (\d+), \d+, (\d+), rkcdev::\w+, (\d+)", rows)}
    have |= {(int(a), int(c), int(d)) for a, c, d in re.findall(
        r"RKC_WAVE_T\([\d.]+, true, (\d+), \d+, (\d+), rkcdev::\w+, (\d+)", rows)}
    text = open(os.path.join(ROOT, "tests", "wave_index_test.cpp")).read()
    line = text[text.index("forms[] = {") + len("forms[] = {"):]
    want = {tuple(int(x) for x in t) for t in re.findall(r"\{(\d+), (\d+), (\d+)\}", line[:line.index(";")])}
    assert have == want and want
