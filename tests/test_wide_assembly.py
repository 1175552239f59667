"""CPU tests: the check that the build makes of the assembly of the dK/dV kernels with 64 keys per wave finds what it looks for, and the build makes it."""
import os
import subprocess
import sys

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02043_amd", "csrc")
sys.path.insert(0, CSRC)
from check_wide import faults  # noqa: E402


def test_the_scan_finds_what_it_looks_for():
    read = "k:\nds_read_b128 v[0:3], v9\n%s\ns_waitcnt lgkmcnt(0)\nv_add_f32 v7, v0, v1\n"
    assert not faults(read % "v_add_f32 v4, v5, v6")
    assert faults(read % "v_mov_b32 v8, v2") and faults(read % "v_mov_b32 v3, v8") and faults(read % "s_waitcnt lgkmcnt(1)\nv_mov_b32 v8, v2")
    around = "k:\nds_read_b128 v[0:3], v9\ns_cbranch_scc1 .L1\ns_waitcnt lgkmcnt(0)\n.L1:\nv_add_f32 v7, v0, v1\n"
    assert faults(around) and not faults(around.replace(".L1:", ".L1:\ns_waitcnt lgkmcnt(0)"))
    assert faults("k:\n.L1:\nds_read_b128 v[0:3], v9\ns_cbranch_scc1 .L1\n")
    mfma = "k:\nv_mov_b32 v4, v9\n%s\nv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n"
    assert faults(mfma % "s_nop 0") and not faults(mfma % "s_nop 1")


@pytest.mark.parametrize("sound", [True, False])
def test_an_unsound_object_is_not_built(tmp_path, sound):
    """The rule of fl_inst_wide.hip, on a kernel that uses what it reads behind the wait, or in front of it."""
    body = 'asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(x) : "v"(8u * threadIdx.x));\n'
    wait = 'asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); __builtin_amdgcn_sched_barrier(0);\n'
    mfma = 'asm volatile("s_nop 1\\n\\tv_mfma_f32_32x32x16_bf16 %0, %1, %1, %0" : "+a"(acc) : "v"(a));\n'
    use = "int y = x[0] * n + x[1]; asm volatile(\"\" : \"+v\"(y)); __builtin_amdgcn_sched_barrier(0);\n"
    (tmp_path / "fl_inst_wide.hip").write_text("""#include <hip/hip_runtime.h>
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
__global__ void k(float* out, i32x4 a, int n) {
i32x2 x; f32x16 acc = {};
%s
for (int r = 0; r < 16; ++r) out[r] = acc[r] + y;
}
""" % (mfma + body + (wait + use if sound else use + wait)))
    r = subprocess.run(["make", "-f", os.path.join(CSRC, "Makefile"), "-C", str(tmp_path), "HDRS=", "HERE=" + CSRC, "PYTHON=" + sys.executable, "_build/fl_inst_wide.o"],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == sound, r.stdout + r.stderr
    assert (tmp_path / "_build" / "fl_inst_wide.o").exists() == sound
    assert sound or "in flight since" in r.stdout
