"""The library's host side when memory runs out: every entry point returns a status.  And what
importing the package leaves alone."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("errors") / "alloc_failures")
    csrc = os.path.join(ROOT, "paper_1711_00244_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-w", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "alloc_failures.cpp")] + [os.path.join(csrc, s) for s in ("compress.cpp", "huffman.cpp", "planner.cpp")] +
                   ["-o", exe], check=True)
    return exe


@pytest.mark.parametrize("what", ["team", "serialize", "deserialize", "compress", "plan"])
def test_every_allocation_may_fail(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)


def test_the_import_leaves_ctypes_pythonapi_alone():
    code = ("import ctypes; f = ctypes.pythonapi.PyBytes_FromStringAndSize; before = f.restype, f.argtypes\n"
            "from paper_1711_00244_amd import binding\n"
            "assert (f.restype, f.argtypes) == before, (f.restype, f.argtypes)")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
