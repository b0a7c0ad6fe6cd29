// Stand-ins for the library and for torch's current stream, linked with native/calls.cpp in place of
// libunstep.so: each entry point counts its calls and returns a status the test sets (no GPU).
#include <c10/hip/HIPStream.h>

#include "unstep.h"

extern "C" {
int stub_calls = 0;         // calls of any entry point that would enqueue work
int stub_fail_next = 0;     // status of the next such call; UNSTEP_OK for the others
const void* stub_handle = nullptr;   // the handle of the last one
const void* stub_pointer = nullptr;  // its cos or sin table if one of them is null, or its log-sum-exp
const void* stub_scratch = nullptr;  // the scratch of the last attention or step
size_t stub_workspace = 0;  // what unstep_attn_workspace_size reports

static int called(const void* handle = nullptr, const void* p = nullptr, const void* p2 = nullptr) {
  ++stub_calls;
  stub_handle = handle;
  stub_pointer = p && p2 ? p : nullptr;
  const int rc = stub_fail_next;
  stub_fail_next = UNSTEP_OK;
  return rc;
}

const char* unstep_last_error(void) { return "the stub's error"; }
int unstep_kv_append(unstep_cache* c, int32_t, int32_t, const void*, const void*, const void*, int64_t, int64_t, const float* cos,
                     const float* sin, void*, void*) {
  return called(c, cos, sin);
}
int unstep_kv_append_qknorm(unstep_cache* c, int32_t, int32_t, const void*, const void*, const void*, int64_t, int64_t,
                            const float* cos, const float* sin, const void*, const void*, double, void*, void*) {
  return called(c, cos, sin);
}
int unstep_attn_workspace_size(const unstep_cache*, int32_t, int32_t, int32_t, size_t* bytes) {
  *bytes = stub_workspace;
  return UNSTEP_OK;
}
int unstep_window_attn(const unstep_cache* c, int32_t, int32_t, int32_t, const void*, void*, float* lse, float, void* ws, size_t, void*) {
  stub_scratch = ws;
  return called(c, lse, lse);
}
int unstep_step(unstep_cache* c, int32_t, int32_t, int32_t, const void*, const void*, const void*, int64_t, int64_t, const float* cos,
                const float* sin, void*, void*, float*, float, void* ws, size_t, void*) {
  stub_scratch = ws;
  return called(c, cos, sin);
}
int unstep_linear(const void*, const void*, const void*, void*, int32_t, int32_t, int32_t, void*) { return called(); }
int unstep_renoise(const void*, const void*, double, void*, int64_t, void*) { return called(); }
int unstep_emit(const void*, const void*, double, void*, int64_t, void*) { return called(); }
}

namespace c10::hip {
HIPStream getCurrentHIPStream(DeviceIndex) {
  return HIPStream(HIPStream::UNCHECKED, Stream(Stream::DEFAULT, Device(DeviceType::HIP, 0)));
}
hipStream_t HIPStream::stream() const { return nullptr; }
}  // namespace c10::hip
