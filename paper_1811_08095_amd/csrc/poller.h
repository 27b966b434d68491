// Host polling of a solve's device scalars, a few iterations behind the GPU: each
// step writes its records into one of four pinned mirrors, an event behind it.
#pragma once
#include "runtime.h"

namespace odwf {

struct Poller {
  hipStream_t st = nullptr;
  CGScal* host = nullptr;  // pinned, 4 slots
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  long k = 0;              // steps pushed
  bool handed = false;     // a mirror was given to a step
  hipError_t init(hipStream_t stream) {
    st = stream;
    HIPRET(hipHostMalloc((void**)&host, 4 * MAXRHS * sizeof(CGScal), hipHostMallocDefault));
    for (int i = 0; i < 4; i++) HIPRET(hipEventCreateWithFlags(&ev[i], hipEventDisableTiming));
    return hipSuccess;
  }
  ~Poller() {
    // every step that was given a mirror writes it until it ends, also one whose
    // event could not be recorded
    if (handed) (void)hipStreamSynchronize(st);
    for (int i = 0; i < 4; i++)
      if (ev[i]) (void)hipEventDestroy(ev[i]);
    if (host) (void)hipHostFree(host);
  }
  // the mirror the next step writes, once its previous contents are complete
  hipError_t next(CGScal** mirror) {
    const int slot = (int)(k % 4);
    if (k >= 4) HIPRET(hipEventSynchronize(ev[slot]));
    *mirror = host + slot * MAXRHS;
    handed = true;
    return hipSuccess;
  }
  hipError_t push() {  // behind that step
    HIPRET(hipEventRecord(ev[k % 4], st));
    k++;
    return hipSuccess;
  }
  // records as of `lag` pushes ago (null if there are none yet)
  hipError_t view(int lag, const CGScal** v) {
    *v = nullptr;
    if (k <= lag) return hipSuccess;
    const int slot = (int)((k - 1 - lag) % 4);
    HIPRET(hipEventSynchronize(ev[slot]));
    *v = host + slot * MAXRHS;
    return hipSuccess;
  }
};

}  // namespace odwf
