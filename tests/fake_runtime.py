"""A stand-in for the HIP runtime, for tests without a GPU of what the library launches: memory is the host's, every call succeeds, kernels do not run, and
the names of those launched are written to a file in order."""
import os
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HAVE = shutil.which("hipcc") is not None

PROPS = r"""
#include <hip/hip_runtime_api.h>
#include <cstring>
extern "C" void fake_properties(void *out)
{
    hipDeviceProp_t p;
    std::memset(&p, 0, sizeof p);
    p.multiProcessorCount = 256;
    std::memcpy(out, &p, sizeof p);
}
"""

RUNTIME = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
struct dim { unsigned x, y, z; };
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> n; return n; }
static dim g_grid, g_block;
static size_t g_lds;
static void *g_stream;
extern "C" {
void fake_properties(void *);
#define SUCCEEDS(f) int f() { return 0; }
SUCCEEDS(hipDeviceSynchronize) SUCCEEDS(hipEventDestroy) SUCCEEDS(hipEventQuery) SUCCEEDS(hipEventRecord) SUCCEEDS(hipEventSynchronize)
SUCCEEDS(hipFuncSetAttribute) SUCCEEDS(hipGetLastError) SUCCEEDS(hipSetDevice) SUCCEEDS(hipStreamDestroy) SUCCEEDS(hipStreamSynchronize)
SUCCEEDS(hipStreamWaitEvent) SUCCEEDS(hipStreamWaitValue64) SUCCEEDS(hipStreamWriteValue64) SUCCEEDS(__hipRegisterVar) SUCCEEDS(__hipUnregisterFatBinary)
int hipDeviceGetAttribute(int *v, int, int) { *v = 8; return 0; }                    // the only one asked for: XCDs
int hipEventCreate(void **e) { *e = e; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = e; return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 0.01f; return 0; }
int hipMalloc(void **p, size_t n) { *p = std::calloc(1, n); return 0; }
int hipExtMallocWithFlags(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
int hipFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = s; return 0; }
int hipExtStreamCreateWithCUMask(void **s, unsigned, const unsigned *) { *s = s; return 0; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevicePropertiesR0600(void *p, int) { fake_properties(p); return 0; }
const char *hipGetErrorString(int) { return "no error"; }
int hipGetSymbolAddress(void **p, const void *) { static char scratch[16 << 20]; *p = scratch; return 0; }
void **__hipRegisterFatBinary(const void *) { static void *one; return &one; }
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
int __hipPushCallConfiguration(dim g, dim b, size_t lds, void *s) { g_grid = g; g_block = b; g_lds = lds; g_stream = s; return 0; }
int __hipPopCallConfiguration(dim *g, dim *b, size_t *lds, void **s) { *g = g_grid; *b = g_block; *lds = g_lds; *s = g_stream; return 0; }
int hipLaunchKernel(const void *f, dim, dim, void **, size_t, void *)
{
    static FILE *log = std::fopen(std::getenv("FAKE_RUNTIME_LOG"), "w");
    std::fprintf(log, "%s\n", names()[f].c_str());
    std::fflush(log);
    return 0;
}
}
"""


def build(tmp):
    """The library to preload; `tmp` is a directory to build it in."""
    sources = []
    for name, text in (("props", PROPS), ("runtime", RUNTIME)):
        sources.append(os.path.join(tmp, name + ".cpp"))
        with open(sources[-1], "w") as f:
            f.write(text)
    lib = os.path.join(tmp, "libfake.so")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-c", sources[0], "-o", sources[0] + ".o"], check=True, capture_output=True)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", sources[1], sources[0] + ".o", "-o", lib], check=True, capture_output=True)
    return lib


def run(lib, tmp, program, **env):
    """Runs a Python program on the stand-in: what it printed, and the kernels launched, one mangled name each."""
    log = os.path.join(tmp, "log")
    open(log, "w").close()
    kept = {k: v for k, v in os.environ.items() if not k.startswith("ECLIP_")}
    out = subprocess.run([sys.executable, "-c", program], cwd=ROOT, check=True, capture_output=True, text=True, timeout=100,
                         env={**kept, "LD_PRELOAD": " ".join([lib] + kept.get("LD_PRELOAD", "").split()), "FAKE_RUNTIME_LOG": log, **env}).stdout
    with open(log) as f:
        return out, f.read().split()
