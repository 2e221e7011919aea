// Device-side helper of the attention kernels: bitmaps of index lists.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

// 64 bits of a bitmap starting at bit `bitpos` (the bitmap must have two readable words after the first one touched)
__device__ __forceinline__ uint64_t window64(const uint32_t* __restrict__ bm, int bitpos) {
    const int w = bitpos >> 5, sh = bitpos & 31;
    const uint32_t a = bm[w], b = bm[w + 1], c = bm[w + 2];
    uint64_t r = ((static_cast<uint64_t>(b) << 32) | a) >> sh;
    if (sh) r |= static_cast<uint64_t>(c) << (64 - sh);
    return r;
}

}  // namespace
