"""The pool of device memory behind the handles (csrc/devmem.cpp), compiled for
the host against a stand-in for the HIP calls it makes: a device of fixed size
that knows whether queued work is still running."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_00501_amd", "csrc")

STUB = r"""
#pragma once
#include <cstddef>
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m);
hipError_t hipMalloc(void** p, size_t n);
hipError_t hipFree(void* p);
hipError_t hipGetDevice(int* d);
hipError_t hipSetDevice(int d);
hipError_t hipMemGetInfo(size_t* a, size_t* t);
hipError_t hipGetLastError();
hipError_t hipDeviceSynchronize();
"""

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include "devmem.hpp"

// one device of TOTAL bytes; the address space is never reused, so a block seen
// again was kept by the pool
static const size_t TOTAL = 1600;  // the pool keeps a sixteenth: 100 bytes
static size_t used = 0;
static std::map<void*, size_t> blocks;
static long waits = 0;
static bool pending = false;
static hipError_t last = hipSuccess;
static char* next = (char*)0x1000;
static bool full = false;  // not even a few bytes are left

hipError_t hipMalloc(void** p, size_t n) {
    const size_t cost = n == 256 ? 0 : n;  // the pool's own probe
    if (used + cost > TOTAL || (full && n == 256)) { *p = nullptr; return last = hipErrorOutOfMemory; }
    *p = next;
    next += 0x1000;
    blocks[*p] = cost;
    used += cost;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!blocks.count(p)) { std::puts("free of an unknown block"); std::exit(1); }
    used -= blocks[p];
    blocks.erase(p);
    pending = false;  // waits for the device
    ++waits;
    return hipSuccess;
}
static hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    const hipStreamCaptureMode was = mode;
    mode = *m;
    *m = was;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMemGetInfo(size_t* a, size_t* t) { *a = TOTAL - used; *t = TOTAL; return hipSuccess; }
hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipDeviceSynchronize() { pending = false; ++waits; return hipSuccess; }

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
using namespace cs;

static int reuse() {  // a kept block goes out again, after a wait, to its size only
    void *a, *b, *c;
    CHECK(dev_alloc(&a, 40) == hipSuccess);
    pending = true;
    dev_free(a);
    CHECK(pending);
    CHECK(dev_alloc(&b, 41) == hipSuccess && b != a);
    CHECK(dev_alloc(&c, 40) == hipSuccess && c == a && !pending);
    const long w = waits;
    dev_free(b);
    dev_free(c);
    CHECK(dev_alloc(&b, 41) == hipSuccess && waits == w + 1);  // one wait serves all blocks freed before it
    CHECK(dev_alloc(&c, 40) == hipSuccess && waits == w + 1);
    return 0;
}
static int bound() {  // at most a sixteenth is kept, the longest-kept blocks go first
    void* p[5];
    for (auto& q : p) CHECK(dev_alloc(&q, 30) == hipSuccess);
    for (void* q : p) dev_free(q);
    CHECK(used == 90 && !blocks.count(p[0]) && !blocks.count(p[1]) && blocks.count(p[4]));
    void* big;
    CHECK(dev_alloc(&big, 101) == hipSuccess);
    dev_free(big);
    CHECK(used == 90);  // larger than the bound: never kept
    for (int i = 1; i <= 40; ++i) {  // changing sizes
        CHECK(dev_alloc(&p[0], i) == hipSuccess);
        dev_free(p[0]);
        CHECK(used <= 100);
    }
    return 0;
}
static int retry() {  // an allocation that fails gets the kept blocks back and is tried again
    void *a, *b;
    CHECK(dev_alloc(&a, 100) == hipSuccess);
    dev_free(a);
    CHECK(used == 100);
    CHECK(dev_alloc(&b, TOTAL - 50) == hipSuccess && used == TOTAL - 50);
    CHECK(hipGetLastError() == hipSuccess);
    CHECK(dev_alloc(&a, 100) == hipErrorOutOfMemory && !a);
    return 0;
}
static int last_lattice() {
    void *a, *b;
    CHECK(dev_alloc(&a, 40) == hipSuccess && dev_alloc(&b, 50) == hipSuccess);
    dev_free(a);
    dev_lattice_created();
    dev_lattice_destroyed();
    CHECK(used == 90);  // one still lives
    dev_lattice_destroyed();
    CHECK(used == 50);
    dev_free(b);
    CHECK(used == 0);  // nothing is kept without a lattice
    return 0;
}
static int failed_wait() {  // no error is left for the caller's next launch check
    void *a, *b;
    CHECK(dev_alloc(&a, 40) == hipSuccess);
    dev_free(a);
    full = true;
    pending = true;
    CHECK(dev_alloc(&b, 40) == hipSuccess && b != a);
    CHECK(hipGetLastError() == hipSuccess);
    return 0;
}
static int wait() {  // by the probe's free, else by returning kept blocks, else by the device itself
    void *a, *b;
    CHECK(dev_alloc(&a, 40) == hipSuccess && dev_alloc(&b, 50) == hipSuccess);
    for (int k = 0; k < 3; ++k) {
        full = k > 0;
        if (k == 1) dev_free(b);
        pending = true;
        dev_wait(a);
        CHECK(!pending && hipGetLastError() == hipSuccess && mode == hipStreamCaptureModeGlobal);
    }
    CHECK(used == 40);
    dev_wait(nullptr);
    return 0;
}
static int release() {
    void *a, *b;
    CHECK(dev_alloc(&a, 40) == hipSuccess && dev_alloc(&b, 50) == hipSuccess);
    dev_free(a);
    CHECK(used == 90);
    dev_release();
    CHECK(used == 50 && !blocks.count(a) && blocks.count(b));
    dev_release();
    return 0;
}

int main(int, char** v) {
    dev_lattice_created();
    struct { const char* name; int (*f)(); } all[] = {
        {"reuse", reuse}, {"bound", bound}, {"retry", retry}, {"last_lattice", last_lattice}, {"failed_wait", failed_wait},
        {"wait", wait},
        {"release", release},
    };
    for (auto& t : all)
        if (!std::strcmp(t.name, v[1])) return t.f();
    return 2;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("devmem")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "devmem")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", str(d), "-I", CSRC, str(d / "main.cpp"),
                    os.path.join(CSRC, "devmem.cpp"), "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("case", ["reuse", "bound", "retry", "last_lattice", "failed_wait", "wait", "release"])
def test_pool(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
