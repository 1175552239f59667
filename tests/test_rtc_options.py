"""CPU test: the scheduler option that the library gives hipRTC for some run-time compiled variants reaches no other compilation of
the process, neither the next one nor one that another thread has under way."""
import ctypes
import threading

SOURCE = b"""
extern "C" __global__ void k(const float* a, const int* idx, float* o, int n) {
  int t = blockIdx.x * 256 + threadIdx.x;
  float s[32], x = 0.f;
#pragma unroll
  for (int r = 0; r < 32; ++r) s[r] = a[idx[(t * 32 + r) % n]] * (float)r + a[(t * 7 + r * r) % n];
#pragma unroll
  for (int r = 0; r < 32; ++r) x += __expf(s[r]) * s[(r * 5) & 31];
  o[t] = x;
}
"""
OPTION = [b"-mllvm", b"-amdgpu-sched-strategy=iterative-ilp"]


def code_object(options):
    rtc = ctypes.CDLL("libhiprtc.so")
    prog = ctypes.c_void_p()
    assert rtc.hiprtcCreateProgram(ctypes.byref(prog), SOURCE, b"k.hip", 0, None, None) == 0
    opts = [b"--offload-arch=gfx950", b"-O3"] + options
    assert rtc.hiprtcCompileProgram(prog, len(opts), (ctypes.c_char_p * len(opts))(*opts)) == 0
    n = ctypes.c_size_t()
    assert rtc.hiprtcGetCodeSize(prog, ctypes.byref(n)) == 0
    code = ctypes.create_string_buffer(n.value)
    assert rtc.hiprtcGetCode(prog, code) == 0
    rtc.hiprtcDestroyProgram(ctypes.byref(prog))
    return code.raw


def test_option_stays_with_its_compilation():
    from paper_2511_02043_amd import binding as fb
    fb.lib()                                         # (brings hipRTC into the process)
    plain, ilp = code_object([]), code_object(OPTION)
    assert plain != ilp and code_object([]) == plain
    got = {"plain": [], "ilp": []}
    threads = [threading.Thread(target=lambda n=n, o=o: got[n].extend(code_object(o) for _ in range(3)))
               for n, o in (("plain", []), ("ilp", OPTION), ("plain", []))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got["plain"] == [plain] * 6 and got["ilp"] == [ilp] * 3
