// A sum that carries what its last addition rounded off (W. Kahan, "Further remarks on reducing truncation errors", 1965).
#pragma once

// sum += v.  lost: 0 before the first, then what the last addition added too much.  An infinite sum has none: inf - inf
// is NaN, and the sum would be NaN from the next addition on.
__device__ __forceinline__ void compensated_add(float v, float& sum, float& lost) {
  const float x = v - lost, s = sum + x, l = (s - sum) - x;
  lost = fabsf(l) < __builtin_inff() ? l : 0.f;
  sum = s;
}
