#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>
#include <cstring>

namespace hip_host {
extern std::atomic<int> capturing;  // what hipStreamIsCapturing answers
bool inside_one_allocation(const void* first, const void* end);
size_t live_allocations();
}  // namespace hip_host
