"""The pinned result slots against a HIP runtime of stubs (no GPU): a failed call
gives its slot back once its stream was waited for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1608_00263_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "internal.h"
static hipError_t g_wait = hipSuccess, g_query = hipSuccess;
static hipStreamCaptureStatus g_cap = hipStreamCaptureStatusNone;
static int g_waits = 0;
extern "C" {
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { g_waits++; return g_wait; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) { *c = g_cap; return g_query; }
}
using svi::ResultSlot;
static int free_slots() {   // takes what is there and gives it back
    std::vector<ResultSlot *> v;
    for (;;) {
        ResultSlot *s = new ResultSlot(8, nullptr);
        if (!s->ptr) { delete s; break; }
        v.push_back(s);
    }
    const int n = (int)v.size();
    for (ResultSlot *s : v) { s->release(); delete s; }
    return n;
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    CHECK(free_slots() == ResultSlot::COUNT);
    { ResultSlot big(ResultSlot::BYTES + 1, nullptr); CHECK(!big.ptr); }
    g_waits = 0;
    for (int i = 0; i < 40; i++) { ResultSlot s(64, nullptr); CHECK(s.ptr); s.release(); }
    CHECK(g_waits == 0);   // the caller had waited
    for (int i = 0; i < 40; i++) { ResultSlot s(64, nullptr); CHECK(s.ptr); }   // calls that failed after a launch
    CHECK(g_waits == 40 && free_slots() == ResultSlot::COUNT);
    g_wait = hipErrorUnknown;   // nothing known about the kernel: the slot stays out
    { ResultSlot s(64, nullptr); CHECK(s.ptr); }
    g_wait = hipSuccess;
    CHECK(free_slots() == ResultSlot::COUNT - 1);
    g_wait = hipErrorStreamCaptureUnsupported;   // under capture: out while a graph may still come of it
    g_cap = hipStreamCaptureStatusActive;
    { ResultSlot s(64, nullptr); CHECK(s.ptr); }
    CHECK(free_slots() == ResultSlot::COUNT - 2);
    g_cap = hipStreamCaptureStatusInvalidated;   // none will: its kernels never run
    for (int i = 0; i < 40; i++) { ResultSlot s(64, nullptr); CHECK(s.ptr); }
    CHECK(free_slots() == ResultSlot::COUNT - 2);
    g_query = hipErrorUnknown;
    { ResultSlot s(64, nullptr); CHECK(s.ptr); }
    CHECK(free_slots() == ResultSlot::COUNT - 3);
    std::printf("ok\n");
    return 0;
}
"""


def test_failed_calls_give_their_slot_back(tmp_path):
    src, exe = tmp_path / "slots_test.cpp", tmp_path / "slots_test"
    src.write_text(HARNESS)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(rocm, "include"), str(src), os.path.join(CSRC, "slots.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
