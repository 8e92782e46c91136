"""The page-locked buffers that a thread's calls share: what a call that ended
early left in flight is waited for before either buffer is written or freed."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))

STAND_IN = """
#pragma once
#include <cstdio>
#include <cstdlib>
typedef int hipError_t;
typedef void* hipEvent_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
inline int note(char c) { std::putchar(c); return hipSuccess; }
inline int hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return note('A'); }
inline int hipHostFree(void* p) { std::free(p); return note('F'); }
inline int hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (void*)1; return note('C'); }
inline int hipEventRecord(hipEvent_t, hipStream_t) { return note('R'); }
inline int hipEventSynchronize(hipEvent_t) { return note('W'); }
inline int hipStreamSynchronize(hipStream_t) { return note('S'); }
"""


def test_waits_before_it_frees(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STAND_IN)
    exe = str(tmp_path / "stage_order")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", str(tmp_path), "-o", exe,
                           os.path.join(HERE, "stage_order.cpp")])
    out = subprocess.run([exe], stdout=subprocess.PIPE, check=True, timeout=60).stdout.decode()
    assert [tuple(l.split()) for l in out.split("\n") if l] == [
        ("first", "AA"), ("again",), ("early", "CR"),
        ("results", "WFA"),        # waited for, then freed and grown
        ("upload", "FA"), ("early", "R"), ("upload", "WFA")]
