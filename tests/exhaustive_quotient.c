/* The conversion kernels' quotient against the division, exhaustively: for every fp16 mantissa of the scale s and every
 * fp32 mantissa of y, with r = RN(1 / s) and fused steps,
 *     q = RN(y r),  t = RN(q + RN(y - q s) r)    equals    RN(y / s),
 * and r itself from an approximation one unit in the last place off either way, corrected by one step.  (Markstein's
 * correction: P. Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor", 1990.)
 * Powers of two in y and s change nothing while no step leaves the normal range.
 * Build: gcc -O3 -mfma -mavx2 -ffp-contract=off -shared -fPIC.  Returns the number of differences among 2^33 pairs. */
#include <math.h>
#include <stdint.h>
#include <string.h>

static float from_bits(uint32_t u) {
  float f;
  memcpy(&f, &u, 4);
  return f;
}

long long check_scales(int lo, int hi) {   /* fp16 mantissas [lo, hi) */
  long long wrong = 0;
  for (int i = lo; i < hi; ++i) {
    const float s = from_bits(0x3F800000u | ((uint32_t)i << 13)), r = 1.0f / s;
    for (int d = -1; d <= 1; ++d) {
      uint32_t u;
      memcpy(&u, &r, 4);
      const float r0 = from_bits(u + (uint32_t)d);
      if (fmaf(fmaf(-s, r0, 1.0f), r0, r0) != r) ++wrong;
    }
    int bad = 0;
    for (uint32_t m = 0; m < 1u << 23; ++m) {
      const float y = from_bits(0x3F800000u | m);
      const float q = y * r;
      const float t = fmaf(fmaf(-q, s, y), r, q);
      bad += t != y / s;
    }
    wrong += bad;
  }
  return wrong;
}
