"""The decay's exponential on the device, for every fp32 argument, against the double
exp rounded once: tests/exp_check (built by __graft_entry__.build()) as a child process."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu
BINARY = os.path.join(os.path.dirname(os.path.abspath(__file__)), "exp_check")


def test_exp_for_every_value():
    assert os.path.exists(BINARY), "tests/exp_check is missing: run __graft_entry__.build()"
    r = subprocess.run([BINARY], capture_output=True, text=True, timeout=120)
    print(r.stdout, r.stderr, flush=True)
    assert r.stdout.split() == ["exp", str(2 ** 32), "0"], r.stdout
    assert r.returncode == 0
