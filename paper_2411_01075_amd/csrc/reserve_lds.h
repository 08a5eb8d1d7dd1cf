// Dynamic LDS above the default limit has to be allowed per kernel, once.
#pragma once
#include <atomic>
#include "common.h"

namespace cephalo {

// Allows kernel KERN `bytes` of dynamic LDS (the same number in every call).  The flag belongs to the kernel itself, not to its type: kernels
// of one signature need different sizes.  It is set when the attribute is, so a thread that finds it set may launch; two that find
// it clear both set the attribute, to the same value; a failure is tried again by the next launch.
template <auto KERN>
int reserve_lds(const char* who, size_t bytes) {
  static std::atomic<bool> done{false};
  if (done.load(std::memory_order_acquire)) return CEPHALO_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
    return fail(CEPHALO_EHIP, "%s: cannot reserve %zu B of LDS", who, bytes);
  done.store(true, std::memory_order_release);
  return CEPHALO_OK;
}

}  // namespace cephalo
