"""The launches of one call that share a workspace buffer are enqueued
together (CPU only).  A plan with K slices on the direct-load kernel enqueues
two kernels, one that fills the buffer's slots and one that sums them; calls
from several host threads on one stream share the buffer, so another call's
launch -- or the growth of the buffer -- between the two would sum the wrong
slots.  A child process loads a recorder in place of the HIP runtime calls the
library makes (the launches wait a little, so that threads do interleave where
they may), calls from two threads, and checks the recorded order."""
import json
import os
import subprocess
import sys

import pytest

import paper_1607_00145_amd as g

RECORDER = r"""
#include <chrono>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <thread>
struct Dim { uint32_t x, y, z; };
static std::mutex m;
static struct { int thread; char what; } events[4096];
static int n = 0;
static thread_local int self = 0;
static void record(char what) {
    { std::lock_guard<std::mutex> l(m); if (n < 4096) events[n++] = {self, what}; }
    std::this_thread::sleep_for(std::chrono::milliseconds(3));
}
static thread_local Dim grid, block; static thread_local size_t shared; static thread_local void *str;
extern "C" {
void recorder_thread(int i) { self = i; }
int recorder_event(int i, char *what) { if (i >= n) return -1; *what = events[i].what; return events[i].thread; }
int __hipPushCallConfiguration(Dim g, Dim b, size_t s, void *t) { grid = g; block = b; shared = s; str = t; return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *s, void **t) { *g = grid; *b = block; *s = shared; *t = str; return 0; }
int hipLaunchKernel(const void *, Dim, Dim, void **, size_t, void *) { record('L'); return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipStreamIsCapturing(void *, int *c) { *c = 0; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipMalloc(void **p, size_t) { record('M'); *p = (void *)0x7000000000; return 0; }
int hipFree(void *) { record('F'); return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x7100000000; return 0; }
}
"""

CHILD = r"""
import ctypes, json, os, sys, threading
rec = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)   # before the library: its HIP calls bind here
import paper_1607_00145_amd as g
rec.recorder_event.argtypes = [ctypes.c_int, ctypes.POINTER(ctypes.c_char)]
entry = getattr(g, sys.argv[2])
os.environ["GETT_FORCE_TILE"] = "4"   # 128 x 128 x 32, which carries the direct-load kernel
def plan(slices):
    os.environ["GETT_FORCE_KSLICES"] = str(slices)
    st, h = g.gett_plan(0, "a,b", [384, 376], None, "a,c,d", [384, 376, 384], None, "d,b,c",
                        [384, 376, 376], None, 0)
    assert st == 0
    return h, json.loads(g.gett_plan_describe(h))
# thread 0 repeats one plan, thread 1 plans that need ever larger buffers
small, d = plan(16)
grow = [plan(p) for p in (28, 56, 112)]
start = threading.Barrier(2)
def work(i):
    rec.recorder_thread(i)
    start.wait()
    base = (i + 1) << 32
    for r in range(12):
        h = small if i == 0 else grow[r // 4][0]
        st = entry(h, 1.0, base, base + (1 << 30), 0.0, base + (2 << 30), 16)
        assert st == 0, st
ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
[t.start() for t in ts]; [t.join() for t in ts]
ev, what = [], ctypes.c_char()
while (t := rec.recorder_event(len(ev), ctypes.byref(what))) >= 0:
    ev.append([t, what.value.decode()])
print(json.dumps({"events": ev, "kslices": [d["kslices"]] + [x["kslices"] for _, x in grow],
                  "bytes": [x["workspace_bytes"] for _, x in grow]}))
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    d = tmp_path_factory.mktemp("recorder")
    src, lib = d / "recorder.cpp", d / "recorder.so"
    src.write_text(RECORDER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", str(src), "-o",
                    str(lib)], check=True)
    return str(lib)


@pytest.mark.parametrize("entry,launches", [("gett_contract", 2), ("gett_contract_noalloc", 3)])
def test_a_calls_launches_stay_together(recorder, entry, launches):
    """Two launches per call (the slices and their sum), in front of them the
    kernel that clears the counters of the fixed buffer.  Nothing of the other
    thread's -- launch, allocation or release -- falls between them."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(g.__file__)))
    env = dict(os.environ, PYTHONPATH=root)
    r = subprocess.run([sys.executable, "-c", CHILD, recorder, entry], env=env, cwd=root,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    out = json.loads(r.stdout.splitlines()[-1])
    assert min(out["kslices"]) > 1 and max(out["bytes"]) <= 64 << 20
    ev = out["events"]
    assert sum(w == "L" for _, w in ev) == 2 * 12 * launches
    i = 0
    while i < len(ev):
        if ev[i][1] != "L":
            i += 1
            continue
        group = ev[i:i + launches]
        assert len({t for t, _ in group}) == 1 and all(w == "L" for _, w in group), (i, ev)
        i += launches
