// Division of a sum of differences by a count of rows, without the division's long sequence.
#pragma once
#include <cmath>

#ifdef __HIPCC__
#define BDDMP_BOTH __host__ __device__ __forceinline__
#else
#define BDDMP_BOTH inline
#endif

namespace bddmp {

// s / n for a row count n <= 64, with r = 1 / n rounded: s * r, corrected once by the exact remainder
// (Markstein's method), is the correctly rounded quotient while nothing underflows or overflows, which a test
// confirms for every mantissa and n; the division itself elsewhere. (A negative zero gives a positive one.)
BDDMP_BOTH float over_count(float s, float n, float r) {
  const float a = fabsf(s);
  if (a != 0.0f && !(a >= 0x1p-100f && a <= 0x1p100f)) return s / n;
  const float q = s * r;
  return fmaf(fmaf(-q, n, s), r, q);
}

}  // namespace bddmp
