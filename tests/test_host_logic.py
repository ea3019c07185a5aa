"""Host code of the library on a runtime of host memory (tests/native/
fake_hip.hpp): what it allocates and copies, and what it does when an
allocation fails.  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1101_0876_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = tmp_path_factory.mktemp("host")

    def run(name, *args):
        exe = str(out / name)
        subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "tests", "native", name + ".cpp"), os.path.join(PKG, "libpotts.so"),
                        f"-Wl,-rpath,{PKG}", "-Wl,--allow-shlib-undefined"], check=True)
        return subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True, timeout=120).stdout.split()

    return run


def test_batch_after_a_failed_allocation(program):
    assert program("batch_alloc") == ["runs", "6", "misplaced", "0"]
