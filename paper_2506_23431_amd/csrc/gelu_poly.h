// Logarithm of the normal distribution's lower tail, for GELU: host code without device types, so that it can be checked by
// itself.
#pragma once

// Phi(-a) = 2^-(1 + a P(a)), P of degree 9, fitted by weighted least squares to the least largest error of a Phi(-a) over [0, 8],
// where Phi(-8) is 6e-16.  With the coefficients as they stand here that error is 3.1e-9 (at a = 1.09; 1.6e-10 before they were
// rounded to fp32), evaluated in fp32 3.4e-8.  Relative to Phi(-a) it is 9e-7 up to a = 3, 1e-4 at 5, 0.7 % at 6 and 10 % at 7, where
// a Phi(-a) is 4e-3, 1.4e-6, 6e-9 and 9e-12.
constexpr int GELU_TERMS = 10;
constexpr float gelu_coefficient(int i) {
  constexpr float P[GELU_TERMS] = {1.1511042f, 0.45922282f, 0.052425109f, -0.0069032288f, -5.6824283e-5f,
                                   0.00032017249f, -9.3072435e-5f, 1.4872334e-5f, -1.3470777e-6f, 5.3995802e-8f};
  return P[i];
}
