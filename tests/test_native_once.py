"""One-time work per device under several threads (tests/native/once_test.cpp, CPU)."""
import os
import subprocess

EXE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "_out", "once_test")


def test_once_per_device_waits_and_retries():
    assert os.path.exists(EXE), f"{EXE} missing: run tests/native/build_native.py (or __graft_entry__.build())"
    r = subprocess.run([EXE], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "once_test: ok" in r.stdout, r.stdout + r.stderr
