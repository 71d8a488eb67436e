"""A stand-in for the HIP runtime, for host-side tests of libfgfft.so without a
device: host memory for device memory, kernels that do nothing, and a log of
the launches and of the dynamic-LDS limits set.

It is loaded ahead of the real runtime in a process of its own
(``run_with_fake_hip``), where the library's calls bind to it.
"""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>
struct Dim { unsigned x, y, z; };
static std::mutex mu;
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::vector<std::string>& lines() { static std::vector<std::string> v; return v; }
static thread_local struct { Dim g, b; size_t shm; void* s; } cfg;
static int fail_wait = 0;
static void note(const char* what, const void* f, size_t n, Dim g, Dim b) {
  std::lock_guard<std::mutex> l(mu);
  char buf[160];
  snprintf(buf, sizeof buf, " %zu %u %u %u %u", n, g.x, g.y, g.z, b.x);
  lines().push_back(std::string(what) + " " + names()[f] + buf);
}
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  std::lock_guard<std::mutex> l(mu);
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t shm, void* s) { cfg = {g, b, shm, s}; return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* shm, void** s) {
  *g = cfg.g; *b = cfg.b; *shm = cfg.shm; *s = cfg.s; return 0;
}
int hipLaunchKernel(const void* f, Dim g, Dim b, void**, size_t shm, void*) { note("launch", f, shm, g, b); return 0; }
int hipExtLaunchKernel(const void* f, Dim g, Dim b, void**, size_t shm, void*, void*, void*, int) {
  note("launch", f, shm, g, b);
  return 0;
}
int hipFuncSetAttribute(const void* f, int, int v) { note("limit", f, v, Dim{0, 0, 0}, Dim{0, 0, 0}); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { memset(d, v, n); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipEventCreate(void** e) { *e = (void*)8; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)8; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return fail_wait; }
int hipEventElapsedTime(float* t, void*, void*) { *t = 1.0f; return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)8; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
const char* hipGetErrorString(int) { return "fake"; }
void fake_fail_waits(int code) { fail_wait = code; }
void fake_clear() { lines().clear(); }
size_t fake_log(char* out, size_t cap) {
  std::string s;
  for (auto& l : lines()) s += l + "\n";
  if (out && cap > s.size()) memcpy(out, s.c_str(), s.size() + 1);
  return s.size();
}
}
"""

PRELUDE = r"""
import ctypes, json, os, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2411_16583_amd import fgfft
lib = fgfft.load_library()


class HostPlan:
    def __init__(self, grid, precision=0, law=0):
        self.h = ctypes.c_void_p()
        self.N = grid[0] * grid[1] * grid[2]
        assert lib.fg_plan_create((ctypes.c_int * 3)(*grid), (ctypes.c_double * 3)(1.0, 1.0, 1.0), precision, None,
                                  ctypes.byref(self.h)) == 0
        assert lib.fg_set_law(self.h, law) == 0
        self.bytes = lib.fg_plan_workspace_bytes(self.h)
        self.mem = ctypes.create_string_buffer(self.bytes + 256)
        a = ctypes.addressof(self.mem)
        assert lib.fg_plan_set_workspace(self.h, ctypes.c_void_p(a + (-a) % 256), self.bytes) == 0
        self.field = ctypes.create_string_buffer(9 * 8 * self.N + 256)
        f = ctypes.addressof(self.field)
        self.f = ctypes.c_void_p(f + (-f) % 256)
        assert lib.fg_set_material(self.h, self.f, self.f, self.f, self.f, self.f, 1.0, 1.0, 1.0, 1.0) == 0
        assert lib.fg_set_state(self.h, self.f, self.f, self.f, self.f) == 0


def log():
    n = fake.fake_log(None, 0)
    b = ctypes.create_string_buffer(n + 1)
    fake.fake_log(b, n + 1)
    fake.fake_clear()
    out = []
    for line in b.value.decode().splitlines():
        what, name, *nums = line.split()
        out.append([what, name] + [int(v) for v in nums])
    return out


fake.fake_log.restype = ctypes.c_size_t
fake.fake_log.argtypes = [ctypes.c_char_p, ctypes.c_size_t]
"""


def run_with_fake_hip(tmp_path, body):
    """Run `body` (Python, after PRELUDE; it assigns `result`) in a process
    whose libfgfft.so calls the stand-in; returns `result`."""
    src, so = str(tmp_path / "fake.cpp"), str(tmp_path / "libfakehip.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, src], check=True)
    code = PRELUDE + body + "\nprint('RESULT' + json.dumps(result))\nsys.stdout.flush()\nos._exit(0)\n"
    r = subprocess.run([sys.executable, "-c", code, so, ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout.rsplit("RESULT", 1)[1])
