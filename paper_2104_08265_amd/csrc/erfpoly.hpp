// erf on the range of the raster's window edges by one polynomial (a Chebyshev expansion).
#pragma once

#include <hip/hip_runtime.h>

namespace wct {

// erf(x) = x P(s), s = 2 x^2 / X - 1 in [-1, 1] for |x| <= sqrt(X), X = 4.2^2 / 2 (edges of
// windows up to 4.2 sigma).  P is the Chebyshev expansion of erf(x) / x in s up to degree 22,
// computed from the Maclaurin series in 60-digit arithmetic and rewritten in powers of s:
// the first term left out is below 3e-18 and the coefficients' moduli sum to 1, so the
// error is that of the evaluation, a few 1e-16.  25 multiply-adds and no branch, where the
// library's erf takes several times that and the fluctuation's series 100 to 240 operations.
constexpr double kErfPolyNsigma = 4.2;
constexpr double kErfPolyX = 8.820882;
constexpr double kErfPolyEdge = 2.96999;  // below sqrt(X), above 4.2 / sqrt 2
__host__ __device__ __forceinline__ double erf_poly(double x) {
  constexpr double c[23] = {0.47474863132061196, -0.23051951429446726, 0.15777328722547479,
                            -0.10925448496312597, 0.071094086262387321, -0.042370351732950742,
                            0.022951370896564433, -0.011301471847063635, 0.0050762814068785909,
                            -0.0020897596201071627, 0.00079246514470957712, -0.00027818916961402408,
                            9.0821775702635809e-05, -2.7694094396386005e-05, 7.9181388844990494e-06,
                            -2.1301091719977426e-06, 5.4102130290356051e-07, -1.3032820069867011e-07,
                            2.9747394820835666e-08, -6.3040965411920484e-09, 1.3088560202137948e-09,
                            -3.227895251638094e-10, 6.0761118028891174e-11};
  const double s = fma(x * x, 2.0 / kErfPolyX, -1.0);
  double p = c[22];
#pragma unroll
  for (int k = 21; k >= 0; --k) {
    double ck = c[k];
#if defined(__HIP_DEVICE_COMPILE__)
    // the coefficient is made in scalar registers where it is used: kept live across a
    // caller's loop, the 23 of them would take 46 vector registers
    __asm__ volatile("" : "+s"(ck));
#endif
    p = fma(p, s, ck);
  }
  return x * p;
}

}  // namespace wct
