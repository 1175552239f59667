"""CPU tests of the build rules: the C library and the PyTorch module are separate, and the latter follows its interpreter."""
import os
import subprocess
import sys

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02043_amd", "csrc")


def commands(*args):
    """What make would run to build everything anew."""
    return subprocess.run(["make", "-n", "-B", "-C", CSRC, *args], check=True, capture_output=True, text=True).stdout


def test_default_builds_the_module_for_the_interpreter_it_is_given():
    out = commands("PYTHON=" + sys.executable)
    assert "-o ../libflattn.so" in out and "-o ../_fltorch.so" in out and sys.executable + " -c" in out


@pytest.mark.parametrize("args", [("lib",), ("PYTHON=" + sys.executable + " -I -S",)], ids=["lib", "interpreter_without_torch"])
def test_the_c_library_needs_no_torch(args):
    out = commands(*args)
    assert "-o ../libflattn.so" in out and "-o ../libflbench.so" in out and "_fltorch" not in out
