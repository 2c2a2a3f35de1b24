// Decodes of the two-plane and MXFP4 codes into signed bytes, shared by the single-token
// and the several-token passes.
#pragma once

#include "tq_device.hpp"

namespace tq {

// Free-scale two-plane chunks: the 16 bytes of chunk j hold plane 1's 32 trits in bytes
// 0..7 and plane 2's in bytes 8..15; within a plane's two dwords, dword u, byte b, bit
// pair 2s..2s+1 is column 32j + 16u + 4s + b as a 2-bit two's-complement trit (00 = 0,
// 01 = +1, 11 = -1). Shifting the pair to a byte's top bits and masking leaves 64*t as a
// signed byte, so a plane decodes in one or two bitwise operations per activation dword
// and the byte dot's sum is exactly 64 times the trit dot.
constexpr uint32_t kTopPairs = 0xC0C0C0C0u;

// One plane's 32 trits (dwords w0, w1) as 64t bytes in the order of the activation
// dwords: t[4u + s] = columns 16u + 4s .. 16u + 4s + 3.
__device__ __forceinline__ void unpack64t(uint32_t w0, uint32_t w1, int (&t)[8]) {
  t[0] = int((w0 << 6) & kTopPairs); t[1] = int((w0 << 4) & kTopPairs);
  t[2] = int((w0 << 2) & kTopPairs); t[3] = int(w0 & kTopPairs);
  t[4] = int((w1 << 6) & kTopPairs); t[5] = int((w1 << 4) & kTopPairs);
  t[6] = int((w1 << 2) & kTopPairs); t[7] = int(w1 & kTopPairs);
}

// Doubled e2m1 magnitudes by 3-bit index (exponent, mantissa) and their negatives, as
// byte tables for v_perm (bytes 0..3 in the low word, 4..7 in the high word).
constexpr uint32_t kMxPosLo = 0x03020100u, kMxPosHi = 0x0C080604u;  //  0  1  2  3 |  4  6  8  12
constexpr uint32_t kMxNegLo = 0xFDFEFF00u, kMxNegHi = 0xF4F8FAFCu;  // -0 -1 -2 -3 | -4 -6 -8 -12
// v_perm selectors 8, 10, 9, 11 replicate bit 7 of bytes 1, 5, 3, 7 of {src0, src1}.
constexpr uint32_t kSignSel = 0x0B090A08u;

// Four e2m1 codes as signed doubled integers: magnitude indices in bytes of `idx`
// (0..7), sign bits at bit 7 of the bytes of `sgn`.
__device__ __forceinline__ int mx_dec4(uint32_t idx, uint32_t sgn) {
  const uint32_t pos = __builtin_amdgcn_perm(kMxPosHi, kMxPosLo, idx);
  const uint32_t neg = __builtin_amdgcn_perm(kMxNegHi, kMxNegLo, idx);
  // sgn's bytes 0..3 sit at bytes 1, 5, 3, 7 of {sgn, sgn << 8}: 0xFF where negative
  const uint32_t m = __builtin_amdgcn_perm(sgn, sgn << 8, kSignSel);
  return (int)((neg & m) | (pos & ~m));
}

}  // namespace tq
