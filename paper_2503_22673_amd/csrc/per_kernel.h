// What is kept once per kernel and process, apart from the HIP code so that host tests can compile it.
#pragma once
#include <atomic>
#include <cstdint>

// Devices on which a kernel's dynamic LDS limit has been raised.  The kernel is the template argument and not a value: kernels of one signature are
// values of one type, and a static of the place that raises the limit would be shared by all that pass through it.
template <auto* Kernel> inline std::atomic<uint64_t> smem_devices{0};
