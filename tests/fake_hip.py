"""A stand-in for the HIP runtime under libpwl.so, for CPU tests of its host
code: which device it waits for, what it allocates under stream capture, what
it launches.  Two devices of 256 compute units, "device" memory from the
host's heap, kernels that do nothing; every call that matters is logged.

run(body) compiles it, and executes `body` in a process of its own with
  L           libpwl.so with the binding's signatures, its HIP calls bound to the stand-in
  H           the stand-in: H.hipSetDevice, H.fake_capture(stream, on), H.fake_malloc_limit(bytes)
  log()       the calls since the last log(), oldest first, each a list of words
  result(v)   ends the body; v is what run() returns
"""

import json
import os
import subprocess
import sys

from tests.gpu_util import ROOT

_SOURCE = r"""
#include <cstdarg>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
struct dim3_ { uint32_t x, y, z; };
static std::string g_log;
static int g_dev = 0;
static std::set<void*> g_capturing;
static std::map<const void*, std::string> g_name;
static std::map<void*, size_t> g_size;        // live allocations
static size_t g_limit = ~(size_t)0;
static int g_mode = 0;                        // capture mode: 0 global, 1 thread-local, 2 relaxed
static uintptr_t g_next_stream = 0x1000;
static struct { dim3_ g, b; size_t lds; void* s; } g_cfg;
static void put(const char* f, ...) {
  char b[512]; va_list a; va_start(a, f); vsnprintf(b, sizeof b, f, a); va_end(a); g_log += b; g_log += '\n';
}
extern "C" {
const char* fake_log() { static std::string s; s.swap(g_log); g_log.clear(); return s.c_str(); }
void fake_capture(void* s, int on) { if (on) g_capturing.insert(s); else g_capturing.erase(s); }
void fake_malloc_limit(size_t n) { g_limit = n; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_name[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, void* s) {
  g_cfg.g = g; g_cfg.b = b; g_cfg.lds = lds; g_cfg.s = s; return 0;
}
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* lds, void** s) {
  *g = g_cfg.g; *b = g_cfg.b; *lds = g_cfg.lds; *s = g_cfg.s; return 0;
}
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void**, size_t lds, void* s) {
  put("launch %s %u %u %u %zu %p", g_name[f].c_str(), g.x, g.y, b.x, lds, s); return 0;
}
int hipDeviceGetAttribute(int* v, int attr, int) {
  static int calls = 0;                       // (asked in this order: compute units, LDS bytes)
  (void)attr; *v = (calls++ % 2 == 0) ? 256 : 163840; return 0;
}
int hipGetDevice(int* d) { *d = g_dev; return 0; }
int hipSetDevice(int d) { if (d < 0 || d > 1) return 101; g_dev = d; put("setdevice %d", d); return 0; }
int hipDeviceSynchronize() { put("devicesync %d", g_dev); return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
const char* hipGetErrorString(int) { return "fake error"; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char mem[64]; *p = mem; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)(g_next_stream += 16); return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamIsCapturing(void* s, int* st) { *st = g_capturing.count(s) ? 1 : 0; return 0; }
int hipThreadExchangeStreamCaptureMode(int* m) { int o = g_mode; g_mode = *m; *m = o; return 0; }
static int take(void** p, size_t n) {
  if (n > g_limit) return 2;
  *p = calloc(1, n); g_size[*p] = n; return 0;
}
int hipMalloc(void** p, size_t n) {
  if (!g_capturing.empty() && g_mode != 2) return 900;   // not allowed while a stream captures
  int e = take(p, n); if (!e) put("malloc %p %zu", *p, n); return e;
}
int hipMallocAsync(void** p, size_t n, void* s) {
  int e = take(p, n);
  if (!e) put("%s %p %zu %p", g_capturing.count(s) ? "graphmalloc" : "mallocasync", *p, n, s);
  return e;
}
int hipFree(void* p) { put("free %p %d", p, g_dev); g_size.erase(p); free(p); return 0; }
int hipFreeAsync(void* p, void* s) { put("freeasync %p %d %p", p, g_dev, s); g_size.erase(p); free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); put("copy %zu", n); return 0; }
int hipStreamBeginCapture(void*, int) { return 801; }
int hipStreamEndCapture(void*, void**) { return 801; }
int hipGraphInstantiate(void**, void*, void**, char*, size_t) { return 801; }
int hipGraphLaunch(void*, void*) { return 801; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
size_t fake_live() { return g_size.size(); }
}
"""

_PRELUDE = r"""
import ctypes, json, sys
H = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # ahead of the real runtime in the symbol search
H.fake_log.restype = ctypes.c_char_p
H.fake_malloc_limit.argtypes = [ctypes.c_size_t]
H.fake_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
H.fake_live.restype = ctypes.c_size_t
L = ctypes.CDLL(sys.argv[2])
L.pwl_last_error.restype = ctypes.c_char_p
vp, i32, i64, dbl = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_double
L.pwl_build.argtypes = [i32, vp, i32, dbl, dbl, i32, i32, i32, vp, vp]
L.pwl_rebuild.argtypes = [vp, i32, vp, i32, dbl, dbl, i32, i32, vp]
L.pwl_eval.argtypes = [vp, vp, vp, vp, i64, vp]
L.pwl_eval_backward.argtypes = [vp] * 7 + [i64, vp]
L.pwl_batch_create.argtypes = [vp, i32, vp, vp, vp]
L.pwl_batch_eval.argtypes = [vp] * 4
L.pwl_batch_eval_backward.argtypes = [vp] * 7
L.pwl_kde.argtypes = [vp, i32, vp, vp, i32, i32, i32, i32, vp, vp, vp]
for f in ("pwl_table_free", "pwl_batch_free"):
    getattr(L, f).argtypes, getattr(L, f).restype = [vp], None
def log():
    return [l.split() for l in H.fake_log().decode().splitlines()]
def result(v):
    print("RESULT " + json.dumps(v), flush=True)
    sys.exit(0)
def build(N, func=0, part=1, vals=1, a=-5.0, b=5.0):
    t = vp()
    st = L.pwl_build(func, None, 0, a, b, N, part, vals, None, ctypes.byref(t))
    assert st == 0, (st, L.pwl_last_error())
    return t
A = 4096   # any 16-byte aligned "device" address: the stand-in's kernels touch nothing
def backward(t, n, stream=None):
    return L.pwl_eval_backward(t, None, A, A, None, A, A, n, stream)
def batch(tables, offsets):
    h = (vp * len(tables))(*[t.value for t in tables])
    o = (i64 * len(offsets))(*offsets)
    b = vp()
    st = L.pwl_batch_create(h, len(tables), o, None, ctypes.byref(b))
    assert st == 0, (st, L.pwl_last_error())
    return b
"""


def run(tmp_path, body):
    import paper_1510_02975_amd as P
    from paper_1510_02975_amd import build as B
    if not os.path.exists(P.binding.LIB_PATH):
        B.build()
    src, so, py = (os.path.join(str(tmp_path), n) for n in ("fake_hip.cpp", "libfake_hip.so", "body.py"))
    with open(src, "w") as f:
        f.write(_SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, src], check=True)
    with open(py, "w") as f:
        f.write(_PRELUDE + body)
    r = subprocess.run([sys.executable, py, so, P.binding.LIB_PATH], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    last = [l for l in r.stdout.splitlines() if l.startswith("RESULT ")]
    assert r.returncode == 0 and last, r.stdout[-2000:] + r.stderr[-2000:]
    return json.loads(last[-1][len("RESULT "):])
