// wait_upload (layer_host.h) against stand-ins for the HIP calls that it makes: which calls wait on the device.
#include "layer_host.h"

static int waits = 0, queries = 0;
static bool done = false;
static hipError_t last = hipSuccess;

extern "C" {
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++waits; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) {
  ++queries;
  if (!done) last = hipErrorNotReady;
  return done ? hipSuccess : hipErrorNotReady;
}
hipError_t hipPeekAtLastError() { return last; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
}

#define CHECK(c) if (!(c)) { printf("line %d: %s (waits %d, queries %d)\n", __LINE__, #c, waits, queries); return 1; }

int main() {
  hgnn_graph g;
  hipStream_t one = (hipStream_t)0x2, other = (hipStream_t)0x1000;
  CHECK(hgnn::wait_upload(&g, one) == hipSuccess && waits == 1)
  CHECK(hgnn::wait_upload(&g, one) == hipSuccess && waits == 2)       // the same handle, perhaps another stream
  CHECK(hgnn::wait_upload(&g, other) == hipSuccess && waits == 3)
  CHECK(last == hipSuccess)                                            // "not ready" does not stay behind ...
  last = hipErrorInvalidValue;
  CHECK(hgnn::wait_upload(&g, one) == hipSuccess && waits == 4 && last == hipErrorInvalidValue)   // ... and what was there does
  last = hipSuccess;
  done = true;
  CHECK(hgnn::wait_upload(&g, one) == hipSuccess && waits == 4)
  const int asked = queries;
  CHECK(hgnn::wait_upload(&g, other) == hipSuccess && waits == 4 && queries == asked)   // remembered for every stream
  printf("upload wait ok\n");
  return 0;
}
