// LBP codes (Algorithm 1) of four packed pixels at a time.
#pragma once
#include <cstdint>

#include <hip/hip_runtime.h>

namespace pd {

// Per byte of four packed pixels, n >= c in bit 7 (the other bits are
// don't-care): the low seven bits are compared with the byte's top bit as a
// guard against borrows between bytes, and the top bits decide where they
// differ.
__device__ __forceinline__ uint32_t ge_bytes(uint32_t n, uint32_t c, uint32_t c_low) {
    const uint32_t d = (n | 0x80808080u) - c_low;
    // (n & ~c) | (~(n ^ c) & d) as one three-input bit operation
    return __builtin_amdgcn_bitop3_b32(n, c, d, 0xB2);
}

// Merges the eight comparison words (answer in bit 7 of each byte) into one
// LBP code per byte, neighbour k in bit 7 - k: the bit-reversed order of the
// code Algorithm 1 defines, with which tables of bins are indexed.
__device__ __forceinline__ uint32_t lbp_codes4(const uint32_t (&r)[8]) {
    // (a & m) | (b & ~m) as one three-input bit operation
    auto sel = [](uint32_t m, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA); };
    const uint32_t t01 = sel(0x80808080u, r[0], r[1] >> 1), t23 = sel(0x80808080u, r[2], r[3] >> 1);
    const uint32_t t45 = sel(0x80808080u, r[4], r[5] >> 1), t67 = sel(0x80808080u, r[6], r[7] >> 1);
    const uint32_t q0 = sel(0xC0C0C0C0u, t01, t23 >> 2), q1 = sel(0xC0C0C0C0u, t45, t67 >> 2);
    return sel(0xF0F0F0F0u, q0, q1 >> 4);
}

}  // namespace pd
