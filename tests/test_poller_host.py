"""The host side of a solve's polling when HIP calls fail (CPU only): csrc/poller.h
compiled against a stand-in for the HIP runtime whose calls fail on demand."""
import os
import subprocess

from paper_1811_08095_amd import build_lib

HIP = """
#pragma once
#include <stddef.h>
#include <stdlib.h>
enum hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
typedef struct ihipStream_t* hipStream_t;
typedef struct ihipEvent_t* hipEvent_t;
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
extern int fail_sync, fail_record, stream_syncs, freed_after_sync;
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
inline hipError_t hipHostFree(void* p) { freed_after_sync = stream_syncs; free(p); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return fail_record ? hipErrorUnknown : hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return fail_sync ? hipErrorUnknown : hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { stream_syncs++; return hipSuccess; }
"""

MAIN = """
#include "poller.h"
#include <cstdio>
int fail_sync, fail_record, stream_syncs, freed_after_sync;
#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\\n", __LINE__, #c); return 1; } } while (0)
int main() {
  odwf::CGScal* m = nullptr;
  const odwf::CGScal* v = nullptr;
  {
    odwf::Poller p;
    EXPECT(p.init(nullptr) == hipSuccess);
    for (int i = 0; i < 4; i++) {
      EXPECT(p.next(&m) == hipSuccess && m == p.host + i * odwf::MAXRHS);
      EXPECT(p.push() == hipSuccess);
      EXPECT(p.view(2, &v) == hipSuccess && (i < 2 ? v == nullptr : v == p.host + (i - 2) * odwf::MAXRHS));
    }
    // a wait that fails is an error, not "no mirror" and not "nothing to see yet"
    fail_sync = 1;
    EXPECT(p.next(&m) != hipSuccess);
    EXPECT(p.view(2, &v) != hipSuccess && v == nullptr);
    fail_sync = 0;
    // a step was launched, its event could not be recorded: it still writes its mirror
    EXPECT(p.next(&m) == hipSuccess);
    fail_record = 1;
    EXPECT(p.push() != hipSuccess);
    fail_record = 0;
  }
  EXPECT(stream_syncs == 1 && freed_after_sync == 1);
  { odwf::Poller p; EXPECT(p.init(nullptr) == hipSuccess); }  // no step: nothing to wait for
  EXPECT(stream_syncs == 1);
  return 0;
}
"""


def test_polling_errors_reach_the_caller(tmp_path):
    os.makedirs(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "t")
    subprocess.check_call(["g++", "-std=c++17", "-I" + str(tmp_path), "-I" + build_lib.CSRC,
                           str(tmp_path / "main.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
