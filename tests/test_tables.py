"""The launch tables' argument form, checked on the host: `tables_check.cpp`
packs the plans of launches on both sides of the form's limits and reads every
word back.  And their staging: `staging_check.cpp` runs it against replaced
runtime calls.  Built with hipcc for the host only; no GPU is touched."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_argument_form_round_trip(tmp_path):
    exe = tmp_path / "tables_check"
    src = os.path.join(ROOT, "paper_2609_04774_amd", "csrc")
    build = subprocess.run(
        [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"), "-I", src,
         "-x", "hip", os.path.join(ROOT, "tests", "tables_check.cpp"), os.path.join(src, "plan.cpp"),
         "-o", str(exe)],
        capture_output=True, text=True, timeout=600)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.startswith("ok"), run.stdout + run.stderr


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_staging_slots(tmp_path):
    exe = tmp_path / "staging_check"
    src = os.path.join(ROOT, "paper_2609_04774_amd", "csrc")
    build = subprocess.run(
        [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"), "-I", src,
         "-x", "hip", os.path.join(ROOT, "tests", "staging_check.cpp"), os.path.join(src, "plan.cpp"),
         "-o", str(exe)],
        capture_output=True, text=True, timeout=600)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.startswith("ok"), run.stdout + run.stderr
