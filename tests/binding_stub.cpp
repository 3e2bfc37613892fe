// Stands in for the GPU under the Python binding, for tests on the CPU: the current stream is the
// null stream.
#include <c10/hip/HIPStream.h>

namespace c10::hip {
HIPStream getCurrentHIPStream(DeviceIndex) {
  return HIPStream(HIPStream::UNCHECKED, Stream(Stream::DEFAULT, Device(DeviceType::CUDA, 0)));
}
hipStream_t HIPStream::stream() const { return nullptr; }
}  // namespace c10::hip
