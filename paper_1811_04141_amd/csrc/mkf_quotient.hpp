// mkf_quotient.hpp -- exact quotients by a divisor whose reciprocal is at hand.
#pragma once

#include <math.h>

namespace mkf {

// a / d, inv = 1 / d rounded, d the square root of a positive float (so inv is
// normal, or zero where d is infinite): Markstein's corrected quotient (P. W.
// Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", IBM J. Res. Dev. 34, 1990).  The product with the reciprocal is
// corrected once by its exact remainder, which rounds as the division does, in 5
// instructions instead of the 10 of a general one.  Where the remainder overflows
// (an infinite operand or quotient) the product is already what the division
// gives.  It differs from the division only where the remainder is subnormal (|a|
// < 1e-30), by one ulp at most, and in the sign of a zero from a negative zero.
__host__ __device__ __forceinline__ float over(float a, float d, float inv) {
  const float q = a * inv;
  const float r = fmaf(-q, d, a);
  return fabsf(r) < __builtin_inff() ? fmaf(r, inv, q) : q;
}

}  // namespace mkf
