"""The library's host code with the HIP calls defined by a test program
(tests/fake_device/driver.cpp): no GPU is needed.

- grids: the launches of calls on very large inputs stay within the limits of a
  grid (65,536 in y and z, 2^32 work-items in x).
- kept: after a staging buffer that could not be replaced, the count of the last
  lift is not read from the freed one.
- noalloc: the allocation-free entry point takes every query that fitted its fixed
  array when that was set, and refuses larger ones."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2601_04185_amd", "libimloc.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="libimloc.so is not built")
@pytest.mark.parametrize("test", ["grids", "kept", "noalloc"])
def test_host_code(tmp_path, test):
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "fake_device", "driver.cpp"), LIB, "-Wl,-rpath," + os.path.dirname(LIB),
                    "-Wl,--allow-shlib-undefined", "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe, test], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failure(s)" in r.stdout, r.stdout + r.stderr
