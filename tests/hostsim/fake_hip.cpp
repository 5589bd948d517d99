// A HIP runtime and kernel launchers that only take notes, so that the host
// code of the library (pda_host.cpp) runs whole on a CPU: the launches it makes
// and the arguments it gives them, its workspace, what it does in a capture or
// when an allocation fails. One device of 256 compute units; streams are any
// non-null pointers.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>

#include "pda_internal.h"

namespace {
unsigned long long g_capture = 0;  // id of the capture every stream records into, 0: none
int64_t g_limit = -1;              // allocations above this many bytes fail (-1: none does)
std::map<void*, size_t> g_sizes;
char g_scratch[pda::kShortCountBytes + pda::kScratchBytes];
pda::DecodeArgs g_decode;
pda::PrefillArgs g_prefill;
int g_launches = 0;
int64_t g_last = 0;
}  // namespace

extern "C" {
void sim_reset(unsigned long long capture, int64_t limit) {
  g_capture = capture;
  g_limit = limit;
  g_launches = 0;
}
int sim_launches(void) { return g_launches; }
// the last decode launch
void sim_decode(int64_t* out) {
  out[0] = g_decode.short_parts;
  out[1] = g_decode.short_clear;
  out[2] = g_decode.short_epoch;
  out[3] = (int64_t)g_decode.hdr;
}
// the last prefill launch
void sim_prefill(int64_t* out) {
  out[0] = g_prefill.slots;
  out[1] = (int64_t)g_prefill.v_img;
  out[2] = (int64_t)g_prefill.k_img;
  out[3] = g_prefill.img_tiles;
  out[4] = g_prefill.list_max;
  out[5] = (int64_t)g_prefill.hdr;
  out[6] = (int64_t)g_prefill.items;
  out[7] = (int64_t)g_prefill.parts;
  out[8] = (int64_t)g_prefill.splits;
  out[9] = (int64_t)g_prefill.part_ml;
  out[10] = (int64_t)g_prefill.part_acc;
}
// bytes of the last allocation
int64_t sim_allocated(void) { return g_last; }
// usable bytes from p to the end of its allocation, -1 if it lies in none
int64_t sim_room(int64_t p) {
  for (auto& [base, size] : g_sizes)
    if (p >= (int64_t)base && p <= (int64_t)base + (int64_t)size) return (int64_t)base + (int64_t)size - p;
  return -1;
}

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(static_cast<void*>(p), 0, sizeof *p);
  p->multiProcessorCount = 256;
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (g_limit >= 0 && (int64_t)n > g_limit) return hipErrorOutOfMemory;
  if (g_capture) return hipErrorStreamCaptureUnsupported;
  if (!(*p = std::calloc(1, n))) return hipErrorOutOfMemory;
  g_sizes[*p] = n;
  g_last = (int64_t)n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  g_sizes.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t, hipStreamCaptureStatus* s, unsigned long long* id) {
  *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  *id = g_capture;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "simulated"; }
}  // extern "C"

namespace pda {
hipError_t launch_decode(const DecodeArgs& a, Variant, KvType, hipStream_t) { return g_decode = a, ++g_launches, hipSuccess; }
hipError_t launch_combine(const DecodeArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_prefix(const DecodeArgs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_append(const AppendArgs&, KvType, hipStream_t) { return ++g_launches, hipSuccess; }
hipError_t launch_prefill(const PrefillArgs& a, KvType, hipStream_t) { return g_prefill = a, ++g_launches, hipSuccess; }
hipError_t decode_occupancy(Variant, KvType, int, int, bool, int* w) { return *w = 8, hipSuccess; }
hipError_t scratch_address(void** p) { return *p = g_scratch, hipSuccess; }
}  // namespace pda
