"""Host-only tests of the device allocator's block pool (pool.hpp): blocks held
for a call's own stream, waits before reuse, and calls on several threads near
the device's capacity."""
import os
import subprocess

import pytest

from tests.test_sched import CSRC, HERE, SANITIZERS


@pytest.mark.parametrize("sanitize", sorted(SANITIZERS))
def test_block_pool(tmp_path, sanitize):
    exe = tmp_path / "pool_driver"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-pthread", *SANITIZERS[sanitize], "-I", CSRC,
                           os.path.join(HERE, "native", "pool_driver.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "FAIL" not in r.stdout and r.stdout.strip().endswith("PASSED")
    assert "Sanitizer" not in r.stderr
