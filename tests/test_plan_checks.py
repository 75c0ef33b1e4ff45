"""The checks of tests/native/plan_checks.hip: libace's host code under
AddressSanitizer and UndefinedBehaviorSanitizer against a stand-in for the HIP
runtime, so that workspace sizes, allocation failures and the reads that a
launch's arguments imply are checked without a GPU
(paper_1601_07159_amd/build.py builds the program)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EXE = os.path.join(ROOT, "tests", "native", "ace_plan_checks")


def test_plan_checks():
    if not os.path.exists(EXE):
        pytest.skip("plan checks not built (paper_1601_07159_amd/build.py)")
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    for k in ("ACE_LOG", "ACE_TUNE", "ACE_TUNE_CACHE"):
        env.pop(k, None)
    r = subprocess.run([EXE], env=env, capture_output=True, text=True, timeout=240)
    print(r.stdout[-8000:])
    print(r.stderr[-8000:])
    assert r.returncode == 0
    assert ", 0 failures" in r.stdout
