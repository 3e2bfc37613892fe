// Stands in for the GPU under the Python binding, for tests on the CPU: the current stream is the
// null stream, and the library's calls that pass data between kernels through scratch memory only
// take their time and notice another call on the same scratch meanwhile.
#include <c10/hip/HIPStream.h>
#include <unistd.h>

#include <atomic>

#include "cure.h"

namespace c10::hip {
HIPStream getCurrentHIPStream(DeviceIndex) {
  return HIPStream(HIPStream::UNCHECKED, Stream(Stream::DEFAULT, Device(DeviceType::CUDA, 0)));
}
hipStream_t HIPStream::stream() const { return nullptr; }
}  // namespace c10::hip

namespace {
std::atomic<int> g_overlaps{0}, g_calls{0}, g_inside[4];
cure_status enqueue(int scratch) {
  if (g_inside[scratch].fetch_add(1) > 0) ++g_overlaps;
  usleep(5000);
  --g_inside[scratch];
  ++g_calls;
  return CURE_OK;
}
}  // namespace

extern "C" {
int stub_overlaps() { return g_overlaps; }
int stub_calls() { return g_calls; }

cure_status cure_margins(const void*, int32_t, int32_t, int32_t, int32_t, int64_t, float*, int32_t*, float*,
                         int32_t*, float*, float*, int32_t, float, int32_t, int32_t, int32_t*, int32_t*, void*,
                         size_t, void*) {
  return enqueue(0);
}
cure_status cure_margins_accept(const void*, int32_t, int32_t, int32_t, int32_t, int64_t, float*, int32_t*,
                                float*, int32_t*, float*, float*, int32_t, float, int32_t, int32_t, int32_t*,
                                int32_t*, const int32_t*, const int32_t*, const int32_t*, const int32_t*,
                                int32_t*, int32_t*, int32_t*, int32_t*, int32_t*, void*, size_t, void*) {
  return enqueue(0);
}
cure_status cure_margins_noalloc(const void*, int32_t, int32_t, int32_t, int32_t, int64_t, float*, int32_t*,
                                 float*, int32_t*, float*, float*, int32_t, float, int32_t, int32_t, int32_t*,
                                 int32_t*, void*) {
  return enqueue(1);
}
cure_status cure_tree_attn(const void*, const void*, const void*, void*, float*, int32_t, int32_t, int32_t,
                           int32_t, int32_t, int32_t, float, const int64_t*, const int32_t*, const int32_t*,
                           const int32_t*, int32_t, const int32_t*, const int32_t*, int32_t, uint32_t, int32_t*,
                           void*, size_t, void*) {
  return enqueue(2);
}
cure_status cure_repair_tree(const void*, int32_t, int32_t, int32_t, int32_t, int64_t, const float*,
                             const int32_t*, const int32_t*, const int32_t*, int32_t, int32_t, int32_t, float,
                             int32_t, int32_t, const int32_t*, int32_t, int32_t*, int32_t*, int32_t*, int32_t*,
                             void*, size_t, void*) {
  return enqueue(3);
}
}
