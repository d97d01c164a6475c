// Dynamic LDS limits of kernels that need more than 64 KB.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <mutex>

namespace purify {

// Raises a kernel's dynamic LDS limit above 64 KB once per process (per kernel and size),
// under a lock: solves on several host threads (the server) then never change a kernel's
// attribute while another thread launches or captures it at a size it already allows.
inline std::mutex& lds_limit_mutex() {
    static std::mutex m;
    return m;
}
inline std::map<const void*, size_t>& lds_limit_set() {
    static std::map<const void*, size_t> s;
    return s;
}

template <typename F>
void set_lds_limit(F* f, size_t bytes) {
    if (bytes <= 65536) return;
    const void* k = reinterpret_cast<const void*>(f);
    std::lock_guard<std::mutex> lk(lds_limit_mutex());
    auto& set = lds_limit_set();
    auto it = set.find(k);
    if (it != set.end() && it->second >= bytes) return;
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess) set[k] = bytes;
}

}  // namespace purify
