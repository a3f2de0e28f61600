"""The LDS reads of the one-vector local solves stay inside what the kernel
allocates (no GPU): the check program csrc/plan_check.cpp walks the planner's
envelopes with the kernel's own index rules, among them a natural-order region
whose last block holds long segments beside padding rows."""
import importlib.util
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_local_sweep_reads_stay_inside(tmp_path):
    spec = importlib.util.spec_from_file_location(
        "amsp_build", os.path.join(ROOT, "paper_2606_04864_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    r = subprocess.run([mod.build_plan_check(str(tmp_path / "plan_check"), sanitize=False), "sweep"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "PASSED (0 failures)" in r.stdout, r.stdout + r.stderr
    assert r.stdout.count("ok sweep ") == 10, r.stdout
