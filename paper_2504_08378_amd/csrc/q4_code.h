// The 4-bit code of one weight, shared by both packers; also compiled for the host, where a test goes
// through all pairs of significands.
#pragma once
#include <hip/hip_runtime.h>

// clamp(rint(w / s), -7, 7) + 8 in the low four bits, for fp16 values w and s with |w| <= about 7 s and
// 0 < s < Inf; inv = approximately 1 / s.  The divide is one multiplication and one correction
// step, which give the same result as the correctly rounded quotient: an exact quotient k + 1/2 (a
// tie) is representable, the corrected quotient is within 2^-44 of the exact one before its only
// rounding, so it is hit exactly; any other quotient of two 11-bit significands lies at least 2^-16
// (relative) from k + 1/2, far outside the error.  Adding 1.5 * 2^23 rounds to the nearest integer,
// ties to even, and leaves it in the low bits.  The IEEE divide sequence was what the packers
// waited for: some 25 instructions an element, 28 us of vector issue for 4096 x 11008.
__host__ __device__ __forceinline__ unsigned q4_code(float w, float s, float inv) {
  const float r = w * inv;
  const float q = fmaf(fmaf(-r, s, w), inv, r);
  return __builtin_bit_cast(unsigned, fminf(7.f, fmaxf(-7.f, q)) + 12582920.f) & 15u;
}
