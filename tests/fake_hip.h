// What a test sees of the HIP runtime in fake_hip.cpp.
#pragma once
#include <cstddef>
#include <functional>

namespace fake {
// Called with (dst, src, bytes) after a device-to-host copy: fills in what
// kernels would have left there.
extern std::function<void(void*, const void*, size_t)> on_readback;
void reset();
// Operations given to a stream that did not wait for everything the other
// streams had been given.
long loose_operations();
// Whether the host has waited for all that the stream was given.
bool host_waited_for(void* stream);
}  // namespace fake
