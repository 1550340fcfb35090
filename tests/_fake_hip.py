"""A host-only stand-in for the HIP runtime calls that libhydro.so makes: memory
is host memory, kernels are logged and not run, every event interval takes one
millisecond.  It shows the order and the shapes of the library's runtime calls
without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
static std::string& text() { static std::string s; return s; }
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static void log(const char* what, const void* a, unsigned long long n = 0) {
  char b[512];
  snprintf(b, sizeof(b), "%s %llx %llu\n", what, (unsigned long long)a, n);
  text() += b;
}
struct Call { dim3 grid, block; size_t shm; hipStream_t st; };
static Call call;
extern "C" {
const char* fake_log() { return text().c_str(); }
void fake_clear() { text().clear(); }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) { call = {g, b, s, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = call.grid; *b = call.block; *s = call.shm; *st = call.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t st) {
  log(("launch " + names()[f]).c_str(), st, (unsigned long long)g.x * g.y * g.z);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(n ? n : 1, 1); log("malloc", *p, n); return hipSuccess; }
hipError_t hipFree(void* p) { log("free", p); free(p); return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { memset(p, v, n); log("memset", p, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t st) { memset(p, v, n); log("memsetasync", st, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { log("devsync", nullptr); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st) { log("sync", st); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { memset(p, 0, sizeof(*p)); p->multiProcessorCount = 256; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char mem[1 << 23]; *p = mem; return hipSuccess; }
}
"""
PRELUDE = """
import ctypes, os
fake = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)  # before the library: its runtime calls bind here
fake.fake_log.restype = ctypes.c_char_p
L = ctypes.CDLL({lib!r})
P, D = ctypes.c_void_p, ctypes.c_double
class Spec(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int) for k in ("scheme", "reconstruction", "riemann", "limiter", "flags")] + [("gamma", D)]
def calls():
    out = [l.rsplit(" ", 2) for l in fake.fake_log().decode().splitlines()]
    fake.fake_clear()
    return [(w, int(a, 16), int(n)) for w, a, n in out]
"""


def run(tmp_path, script):
    """Runs script in a fresh interpreter with the stand-in bound to the library."""
    src, so = tmp_path / "fake_hip.cpp", tmp_path / "libfake_hip.so"
    src.write_text(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + rocm + "/include",
                           "-Wno-attributes", str(src), "-o", str(so)])
    lib = os.path.join(ROOT, "paper_1103_3373_amd", "libhydro.so")
    env = {k: v for k, v in os.environ.items() if k != "HYDRO_TUNE_CACHE"}
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(fake=str(so), lib=lib) + script], capture_output=True,
                       text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
