// Copies between HBM and pinned host staging by one work-group.
//
// The host side of every 16-byte vector is aligned (the bytes before the first
// such address and after the last are done one by one); the HBM side may lie
// at any byte address (a global load needs no alignment).  Each work-item
// keeps kDeep vectors in flight: a host-link round trip takes about 2 us and
// an HBM load about 1, so what one work-group moves is bound by the bytes it
// has in flight (256 work-items x 8 x 16 B = 32 KiB), not by the link.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gsys_device.hpp"

namespace gsys_hc {

using namespace gsys;

constexpr uint32_t kDeep = 8;
typedef u32x4 u32x4_u __attribute__((aligned(1)));
__device__ __forceinline__ u32x4 ldg16_any(const uint8_t* p) { return *gp<const u32x4_u>((uint64_t)p); }

// Bytes of [0, n) before the first 16-byte boundary at or after `a`.
__device__ __forceinline__ uint64_t head_bytes(uint64_t a, uint64_t n) {
  return min<uint64_t>(n, (0 - a) & 15);
}

// Work-items 0 .. nt - 1 copy n bytes from HBM to host staging.
__device__ inline void copy_to_host(uint64_t dst, const uint8_t* src, uint64_t n, uint32_t t,
                             uint32_t nt) {
  const uint64_t h = head_bytes(dst, n), nv = (n - h) / 16, tail = h + nv * 16;
  if (t < h) gp<uint8_t>(dst)[t] = gp(src)[t];
  uint64_t i = t;
  for (; i + (kDeep - 1) * (uint64_t)nt < nv; i += kDeep * (uint64_t)nt) {
    u32x4 v[kDeep];
#pragma unroll
    for (uint32_t k = 0; k < kDeep; ++k) v[k] = ldg16_any(src + h + 16 * (i + k * (uint64_t)nt));
#pragma unroll
    for (uint32_t k = 0; k < kDeep; ++k) stg16(dst + h + 16 * (i + k * (uint64_t)nt), v[k]);
  }
  for (; i < nv; i += nt) stg16(dst + h + 16 * i, ldg16_any(src + h + 16 * i));
  if (tail + t < n) gp<uint8_t>(dst)[tail + t] = gp(src)[tail + t];
}

}  // namespace gsys_hc
