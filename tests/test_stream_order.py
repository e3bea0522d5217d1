"""Events and streams of the calls that use two streams, without a GPU: the
library runs in a child process over stand-ins for the HIP calls that it makes
(nothing is launched), which write down every event, wait and launch.

A capture keeps, for each stream, the events recorded on it, and ends by going
through them; destroying an event takes it from the stream that it was last
recorded on alone.  One event recorded on two streams and destroyed while they
are captured is therefore still in the other's list when the capture ends:
each event has one stream.  And what a side stream was given is waited for
before the call's last launch on the caller's stream, and after all that the
caller's stream had been given."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_1905_01330_amd import _lib as L

STUB = r"""
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
typedef struct { uint32_t x, y, z; } dim3_t;
static uintptr_t next_id = 16;
static void say(const char* what, const void* a, const void* b) {
  static FILE* f = 0;
  if (!f) f = fopen(getenv("TN_STUB_LOG"), "w");
  fprintf(f, "%s %lx %lx\n", what, (unsigned long)a, (unsigned long)b);
  fflush(f);
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipEventCreate(void** e) { *e = (void*)(next_id += 16); say("create", *e, 0); return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void* e) { say("destroy", e, 0); return 0; }
int hipEventRecord(void* e, void* s) { say("record", e, s); return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)f; say("wait", e, s); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)(next_id += 16); return 0; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = 0; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipMemcpyAsync(void* d, const void* p, size_t n, int k, void* s) { (void)d; (void)p; (void)n; (void)k; (void)s; return 0; }
static struct { dim3_t g, b; size_t m; void* s; } cfg;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t m, void* s) {
  cfg.g = g;
  cfg.b = b;
  cfg.m = m;
  cfg.s = s;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* m, void** s) {
  *g = cfg.g;
  *b = cfg.b;
  *m = cfg.m;
  *s = cfg.s;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** a, size_t m, void* s) {
  (void)f; (void)g; (void)b; (void)a; (void)m;
  say("launch", 0, s);
  return 0;
}
"""

CHILD = r"""
import ctypes as C, struct, sys
lib = C.CDLL(sys.argv[1])
class T(C.Structure):
    _fields_ = [("data", C.c_void_p), ("dtype", C.c_int32), ("rank", C.c_int32), ("shape", C.c_int64 * 8), ("stride", C.c_int64 * 8)]
at = [1 << 40]
def tensor(shape, dtype=0):
    t = T(at[0], dtype, len(shape))
    at[0] += 1 << 32
    n = 1
    for i in reversed(range(len(shape))):
        t.shape[i], t.stride[i] = shape[i], n
        n *= shape[i]
    return t
def chain(dims, d=2, dtype=0):
    return (T * (len(dims) - 1))(*[tensor((dims[k], d, dims[k + 1]), dtype) for k in range(len(dims) - 1)])
def place(n):
    p = at[0]
    at[0] += (n + (1 << 33)) >> 32 << 32
    return C.c_void_p(p)
lib.tn_last_error.restype = C.c_char_p
def ok(rc):
    assert rc == 0, lib.tn_last_error()
st, size, out = C.c_void_p(8), C.c_size_t(0), place(1 << 20)
what = sys.argv[2]
if what == "gauge":   # sites with and without a Cholesky attempt, of up to and over 2048 rows
    dims = [1, 7, 40, 80, 160, 100, 20, 40, 1]
    psi = (T * 8)(*[tensor((dims[k], 30 if k == 4 else 7, dims[k + 1]), 1) for k in range(8)])
    ok(lib.tn_mps_left_canonicalize_workspace(8, psi, C.byref(size)))
    ok(lib.tn_mps_left_canonicalize(8, psi, out, place(size.value), size, st))
elif what == "inner":   # steps that share launches, larger ones between them
    psi, phi = [chain([1, 40, 50, 3000, 3000, 40, 30, 3000, 50, 20, 1]) for _ in range(2)]
    ok(lib.tn_mps_inner_workspace(10, psi, phi, C.byref(size)))
    ok(lib.tn_mps_inner(10, psi, phi, out, place(size.value), size, 2, st))
elif what == "sweep":
    psi = chain([1, 40, 50, 2000, 2000, 40, 30, 2000, 50, 20, 1])
    mpo = (T * 10)(*[tensor((1 if k == 0 else 3, 1 if k == 9 else 3, 2, 2)) for k in range(10)])
    ok(lib.tn_mps_env_sweep_workspace(10, psi, mpo, C.byref(size)))
    ok(lib.tn_mps_env_sweep(10, psi, mpo, None, None, out, 3, place(size.value), size, 0, st))
else:   # two chains, small and large steps in turn
    dims = [1, 20, 300, 400, 60, 50, 40, 300, 200, 30, 1]
    psi, phi = [(T * 20)(*(list(chain(dims)) + list(chain(dims)))) for _ in range(2)]
    off = (C.c_int32 * 3)(0, 10, 20)
    ok(lib.tn_mps_inner_batched_workspace(2, off, psi, phi, C.byref(size)))
    ws = place(size.value)
    ok(lib.tn_mps_inner_batched_upload(2, off, psi, phi, ws, size, st))
    ok(lib.tn_mps_inner_batched_launch(2, off, psi, phi, out, ws, size, 0, st))
"""


@pytest.mark.parametrize("call", ["gauge", "inner", "sweep", "batch"])
def test_one_stream_an_event(call, tmp_path):
    cc = shutil.which("gcc") or shutil.which("cc")
    if not cc:
        pytest.skip("no C compiler")
    (tmp_path / "stub.c").write_text(STUB)
    stub = tmp_path / "stub.so"
    subprocess.run([cc, "-shared", "-fPIC", "-O1", "-o", str(stub), str(tmp_path / "stub.c")], check=True)
    log = tmp_path / "log"
    env = dict(os.environ, TN_STUB_LOG=str(log))
    env["LD_PRELOAD"] = " ".join(x for x in (os.environ.get("LD_PRELOAD"), str(stub)) if x)
    for name in ("TN_TUNE", "TN_TUNE_CACHE", "TN_LOG"):
        env.pop(name, None)
    subprocess.run([sys.executable, "-c", CHILD, L.LIB_PATH, call], check=True, env=env, timeout=120)
    lines = [x.split() for x in log.read_text().splitlines()]
    lines = [(what, int(a, 16), int(b, 16)) for what, a, b in lines]
    main, launched, recorded, alive = 8, {8: 0}, {}, set()
    seen = {}       # (stream, other): launches of `other` that the stream's later work waits for
    marks = {}      # event: what its record covers
    last_main = max(i for i, x in enumerate(lines) if x[0] == "launch" and x[2] == main)
    for i, (what, ev, stream) in enumerate(lines):
        if what == "create":
            alive.add(ev)
        elif what == "destroy":
            alive.remove(ev)
        elif what == "record":
            assert ev in alive
            assert recorded.setdefault(ev, stream) == stream, "an event recorded on two streams"
            marks[ev] = launched.get(stream, 0)
        elif what == "wait":
            assert ev in marks, "a wait for an event that was not recorded"
            seen[stream, recorded[ev]] = marks[ev]
        else:
            if stream != main:   # only behind a wait for the caller's stream
                assert (stream, main) in seen
            launched[stream] = launched.get(stream, 0) + 1
            if i == last_main:
                for s, n in launched.items():
                    assert s == main or seen.get((main, s), 0) == n, "work of a side stream that is not waited for"
    assert not alive, "events left"
    assert len(launched) == 2, "the case uses one stream only"
