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


@pytest.mark.parametrize("scratch", [False, True], ids=["registers", "scratch"])
def test_stationary_bias_kernels_are_built_without_scratch(tmp_path, scratch):
    """The rule of fl_inst_pair*.hip refuses an instance that the compiler gives scratch memory."""
    body = "float a[64]; for (int i = 0; i < 64; ++i) a[i] = x[i * n]; x[0] = a[n];" if scratch else "x[threadIdx.x] += n;"
    (tmp_path / "fl_inst_pairtest.hip").write_text("#include <hip/hip_runtime.h>\n__global__ void k(float* x, int n) { %s }\n" % body)
    r = subprocess.run(["make", "-f", os.path.join(CSRC, "Makefile"), "-C", str(tmp_path), "HDRS=", "_build/fl_inst_pairtest.o"], capture_output=True, text=True)
    assert (r.returncode != 0) == scratch, r.stdout + r.stderr
    assert (tmp_path / "_build" / "fl_inst_pairtest.o").exists() == (not scratch)


def test_no_vector_instruction_is_written_by_hand():
    """The wait states that a vector instruction needs behind a matrix instruction which reads or writes its destination are kept by the
    compiler, and it does not look into asm statements."""
    import glob
    import re
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        found = re.findall(r'\basm\b(?:\s+volatile)?\s*\(\s*"[^"]*\bv_\w+', open(path).read())
        assert not found, (path, found)
