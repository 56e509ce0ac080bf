"""How cg_solve_batch returns when a HIP call fails part way: with the error, nothing of the solve still
running on the caller's buffers or copying into the thread's state mirror, and no graph left over.

The library runs here against a stand-in for the HIP runtime that queues what is enqueued on a
stream until the stream or an event is waited for, runs no kernels, and fails one chosen call.  It is loaded
first, into the global scope, so the library's HIP calls bind to it (in a process of its own)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <functional>
#include <deque>
#include <string>
struct dim { uint32_t x, y, z; };
struct Stream { std::deque<std::function<void()>> q; bool capturing = false; };
struct Event { Stream* s = nullptr; size_t upto = 0; };
static Stream null_stream;
static size_t done, queued;   // operations in order over all streams
static int execs, fail_at;
static std::string fail_fn;
static Stream* of(void* s) { return s ? (Stream*)s : &null_stream; }
static int failing(const char* fn) { return fail_fn == fn && --fail_at == 0 ? 1 : 0; }
static void add(void* s, std::function<void()> f) {
  if (of(s)->capturing) return;
  of(s)->q.push_back(f);
  ++queued;
}
static void run(Stream* s) {
  for (; !s->q.empty(); s->q.pop_front(), ++done) s->q.front()();
}
extern "C" {
void fake_fail(const char* fn, int nth) { fail_fn = fn; fail_at = nth; }
int fake_pending() { return (int)(queued - done); }
int fake_execs() { return execs; }
static dim g_grid, g_block; static size_t g_lds; static void* g_stream;
int __hipPushCallConfiguration(dim g, dim b, size_t l, void* s) { g_grid = g; g_block = b; g_lds = l; g_stream = s; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* l, void** s) { *g = g_grid; *b = g_block; *l = g_lds; *s = g_stream; return 0; }
void** __hipRegisterFatBinary(const void*) { static void* p; return &p; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int hipLaunchKernel(const void*, dim, dim, void**, size_t, void* s) { add(s, [] {}); return failing("hipLaunchKernel"); }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "stand-in failure"; }
int hipEventCreate(void** e) { *e = new Event; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = new Event; return 0; }
int hipEventDestroy(void* e) { delete (Event*)e; return 0; }
int hipEventRecord(void* e, void* s) { ((Event*)e)->s = of(s); return failing("hipEventRecord"); }
int hipEventSynchronize(void* e) { if (failing("hipEventSynchronize")) return 1; run(((Event*)e)->s); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = new Stream; return 0; }
int hipStreamDestroy(void* s) { delete (Stream*)s; return 0; }
int hipStreamSynchronize(void* s) { run(of(s)); return 0; }
int hipStreamBeginCapture(void* s, int) { if (failing("hipStreamBeginCapture")) return 1; of(s)->capturing = true; return 0; }
int hipStreamEndCapture(void* s, void** g) { of(s)->capturing = false; *g = (void*)1; return failing("hipStreamEndCapture"); }
int hipGraphDestroy(void*) { return 0; }
int hipGraphInstantiate(void** x, void*, void**, char*, size_t) { if (failing("hipGraphInstantiate")) return 1; *x = (void*)1; ++execs; return 0; }
int hipGraphExecDestroy(void*) { --execs; return 0; }
int hipGraphLaunch(void*, void* s) { if (failing("hipGraphLaunch")) return 1; add(s, [] {}); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { add(s, [=] { memset(p, v, n); }); return 0; }
int hipMemcpyAsync(void* d, const void* c, size_t n, int, void* s) {
  if (failing("hipMemcpyAsync")) return 1;
  add(s, [=] { memcpy(d, c, n); });
  return 0;
}
}
"""

CHILD = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import paper_1411_2223_amd as asq
asq.load()
def buf(n):
    b = ctypes.create_string_buffer(n + 256)
    keep.append(b)
    return (ctypes.addressof(b) + 255) & ~255
keep = []
d = asq.asq_gauge_desc((ctypes.c_int * 4)(4, 4, 4, 4), 3, 18, 9 / 8, -1 / 24)
n = asq.asq_gauge_bytes(ctypes.byref(d))
g = ctypes.c_void_p()
assert asq.asq_gauge_create_device(ctypes.byref(d), buf(256 * 576), buf(256 * 576), buf(n), n, None, ctypes.byref(g)) == 0
ncol, m = 2, (ctypes.c_double * 2)(0.1, 0.2)
mode = asq.ASQ_MODE_MIXED32
w = asq.asq_workspace_bytes(g, ncol, mode)
p = asq.asq_cg_params(1e-10, 100, mode, 0.1, 8, 1)
st = (asq.asq_cg_stats * ncol)()
b, x, work = buf(ncol * 128 * 48), buf(ncol * 128 * 48), buf(w)
fail, nth = sys.argv[3], int(sys.argv[4])
for use_graph in (1, 0):
    p.use_graph = use_graph
    fake.fake_fail(fail.encode(), nth)
    rc = asq.cg_solve_batch(g, ncol, m, b, x, work, w, ctypes.byref(p), st, None)
    print(use_graph, rc, fake.fake_pending(), fake.fake_execs(), flush=True)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("hip")
    (d / "fake.cpp").write_text(RUNTIME)
    so = d / "libfake.so"
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "fake.cpp"), "-o", str(so)],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return so


def _solve(runtime, fail, nth):
    env = dict(os.environ, ASQ_TUNE="0")
    r = subprocess.run([sys.executable, "-c", CHILD, str(runtime), ROOT, fail, str(nth)], env=env,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]


# the second copy is that of the first block's states, the third the second block's
@pytest.mark.parametrize("fail,nth", [("hipStreamBeginCapture", 1), ("hipStreamEndCapture", 1),
                                      ("hipGraphInstantiate", 1), ("hipGraphLaunch", 1), ("hipEventRecord", 1),
                                      ("hipEventRecord", 2), ("hipEventSynchronize", 1), ("hipMemcpyAsync", 2),
                                      ("hipMemcpyAsync", 3)])
def test_failed_call_leaves_nothing_in_flight(runtime, fail, nth):
    for use_graph, rc, pending, execs in _solve(runtime, fail, nth):
        reached = use_graph or not ("Graph" in fail or "Capture" in fail)
        assert rc == (-5 if reached else -3)
        assert pending == 0 and execs == 0


def test_solve_without_failures(runtime):
    assert _solve(runtime, "", 0) == [(1, -3, 0, 0), (0, -3, 0, 0)]
