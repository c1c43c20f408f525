"""Encode plans with the options that the library sets for its models
(tests/plan_options_check.cpp), under AddressSanitizer and
UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_00690_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_plans_with_the_library_options(tmp_path):
    exe = str(tmp_path / "plan_options_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer",
           "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall", "-Werror",
           "-I", CSRC, os.path.join(ROOT, "tests", "plan_options_check.cpp"),
           os.path.join(CSRC, "plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr
    counts = {k: int(v) for k, v in (kv.split("=") for kv in r.stdout.split()[1:])}
    assert counts["plans"] == 3000
    assert min(counts["short"], counts["mixed"], counts["forced"]) > 100 and counts["rule"] > 10
