// Bessel functions J0, J1, Y0, Y1 of a real positive argument in FP64, for the
// 2D Green's function (i/4) H0^(1)(k r) and the cell weights of the discrete
// volume integral operator (Sec. II, "the Green's function ... is
// analytically known").
//
// Method (no vendor special-function library):
//  * x >= 25: Hankel's asymptotic expansion
//      H_nu(x) ~ sqrt(2/(pi x)) (P + i Q) e^{i (x - nu pi/2 - pi/4)},
//      P = sum_k (-1)^k a_2k / x^2k, Q = sum_k (-1)^k a_2k+1 / x^2k+1,
//      a_k(nu) = prod_{m=1..k} (4 nu^2 - (2m-1)^2) / (k! 8^k),
//    summed until the terms fall below 1e-18 (the series is enveloping for real
//    x, and at x >= 25 its smallest term is far below double precision).
//  * 0 < x < 25: Miller's backward recurrence J_{k-1} = (2k/x) J_k - J_{k+1}
//    from an even start index N >= x + 40, normalised by
//    J0 + 2 sum_k J_2k = 1, with Neumann's series
//      Y0 = (2/pi)(ln(x/2) + gamma) J0 - (4/pi) sum_k (-1)^k J_2k / k,
//    and its derivative (Y1 = -Y0')
//      Y1 = (2/pi)((ln(x/2) + gamma) J1 - J0/x)
//           + (2/pi) sum_k (-1)^k (J_2k-1 - J_2k+1) / k.
// Host-callable so it can be checked on the CPU against an independent library.
#pragma once

#include <hip/hip_runtime.h>
#include <cmath>

namespace fwi {

__host__ __device__ inline void bessel01(double x, double* j0, double* j1, double* y0, double* y1) {
  const double PI = 3.14159265358979323846;
  const double EULER = 0.57721566490153286061;
  if (x >= 25.0) {
    double P0 = 1.0, Q0 = 0.0, P1 = 1.0, Q1 = 0.0;
    double t0 = 1.0, t1 = 1.0;
    for (int k = 1; k <= 60; ++k) {
      const double f = (double)(2 * k - 1) * (double)(2 * k - 1);
      t0 *= (0.0 - f) / (8.0 * k * x);
      t1 *= (4.0 - f) / (8.0 * k * x);
      // P takes even k with sign (-1)^(k/2); Q takes odd k with sign (-1)^((k-1)/2)
      if (k & 1) {
        const double s = ((k - 1) / 2) & 1 ? -1.0 : 1.0;
        Q0 += s * t0;
        Q1 += s * t1;
      } else {
        const double s = (k / 2) & 1 ? -1.0 : 1.0;
        P0 += s * t0;
        P1 += s * t1;
      }
      if (fabs(t0) < 1e-18 && fabs(t1) < 1e-18) break;
    }
    double s, c;
    sincos(x, &s, &c);
    const double r2 = 0.70710678118654752440;
    const double c0 = (c + s) * r2, s0 = (s - c) * r2;     // chi = x - pi/4
    const double c1 = (s - c) * r2, s1 = -(s + c) * r2;    // chi = x - 3 pi/4
    const double amp = sqrt(2.0 / (PI * x));
    *j0 = amp * (P0 * c0 - Q0 * s0);
    *y0 = amp * (P0 * s0 + Q0 * c0);
    *j1 = amp * (P1 * c1 - Q1 * s1);
    *y1 = amp * (P1 * s1 + Q1 * c1);
    return;
  }
  const int N = 2 * ((int)x + 20);  // even, >= x + 40
  double fp = 0.0, fc = 1.0;        // f_{k+1}, f_k with k = N
  double S = 2.0 * fc;              // J0 + 2 sum J_2k (N even)
  double sy0 = (((N / 2) & 1) ? -1.0 : 1.0) * fc / (N / 2);
  double sy1 = 0.0;
  double fodd = 0.0;                // f_{m+2} for odd m (f_{N+1} = 0)
  double f1 = 0.0;
  for (int k = N; k >= 1; --k) {
    const double fm = (2.0 * k / x) * fc - fp;
    fp = fc;
    fc = fm;
    const int m = k - 1;
    if (m & 1) {
      const int kk = (m + 1) / 2;
      sy1 += ((kk & 1) ? -1.0 : 1.0) * (fc - fodd) / kk;
      fodd = fc;
      if (m == 1) f1 = fc;
    } else if (m >= 2) {
      S += 2.0 * fc;
      sy0 += (((m / 2) & 1) ? -1.0 : 1.0) * fc / (m / 2);
    } else {
      S += fc;
    }
    if (fabs(fc) > 1e250) {
      const double sc = 1e-250;
      fc *= sc; fp *= sc; fodd *= sc; f1 *= sc; S *= sc; sy0 *= sc; sy1 *= sc;
    }
  }
  const double J0 = fc / S, J1 = f1 / S;
  const double lg = log(0.5 * x) + EULER;
  *j0 = J0;
  *j1 = J1;
  *y0 = (2.0 / PI) * lg * J0 - (4.0 / PI) * sy0 / S;
  *y1 = (2.0 / PI) * (lg * J1 - J0 / x) + (2.0 / PI) * sy1 / S;
}

// H0^(1)(x) = J0 + i Y0 of real x > 0 for the field kernels, which evaluate it
// once per grid point and element (bessel01's recurrence of about x + 40 steps
// and its term-by-term expansion bound them: 221 us per frequency at 256^2 with
// 64 elements, where the stores take 14; 36 with the forms below, bound by
// their FP64 arithmetic).
//  * x < 4: J0 and the regular part Y0 - (2/pi) ln(x/2) J0 as polynomials in x^2;
//  * x >= 4: H0 = sqrt(2/(pi x)) (P + i Q/x) e^{i (x - pi/4)}, P and Q as
//    polynomials in 1/x^2 on [4, 8] and [8, inf).
// Each polynomial is the truncated Chebyshev series of its function on its
// interval (first term left out below 2^-55 of the largest), in powers of the
// interval's variable s in [-1, 1]; the functions themselves were evaluated to
// 50 digits from their series and expansions. Error against 50 digits below
// 6e-16 |H0| plus the rounding of x in the phase, as bessel01's.
template <int N>
__host__ __device__ inline double horner(const double (&a)[N], double s) {
  double v = a[N - 1];
#pragma unroll
  for (int k = N - 2; k >= 0; --k) v = fma(v, s, a[k]);
  return v;
}
__host__ __device__ inline void hankel0(double x, double* j0, double* y0) {
  constexpr double kJ0[14] = {
      -1.965480952704682e-1, -5.65959973761085006e-1, 4.79528082151010703e-1, -1.31032063513645467e-1,
      1.83527006100656499e-2, -1.57895413668797297e-3, 9.22817399022653375e-5, -3.91034197870673673e-6,
      1.25772806293626957e-7, -3.17743951371879604e-9, 6.47443023732125842e-11, -1.08683733822377686e-12,
      1.52998319632434314e-14, -1.83079044195994749e-16};
  constexpr double kB0[14] = {
      4.71652905076182966e-1, -1.98814148740716849e-1, -1.92095175873352418e-1, 9.25758139948608019e-2,
      -1.65615972388590062e-2, 1.65495797465905129e-3, -1.07492925779080639e-4, 4.9366451720794115e-6,
      -1.69356334495843359e-7, 4.51332528391887196e-9, -9.62365583489981785e-11, 1.68028819133182185e-12,
      -2.44871053026223326e-14, 3.02174056343150012e-16};
  constexpr double kP4[16] = {
      9.97399301828614183e-1, -1.48450160424359661e-3, 4.00551814717931949e-5, -2.66063743759658328e-6,
      2.83593225985800402e-7, -4.05424782421050271e-8, 7.08332921752134666e-9, -1.43223310110110185e-9,
      3.23638317410567204e-10, -7.98562171915462067e-11, 2.13557247277196223e-11, -6.03773034101528846e-12,
      1.56391184619718856e-12, -4.60959257605373175e-13, 2.83494347319774311e-13, -9.96647697924271307e-14};
  constexpr double kQ4[18] = {
      -1.22415190620664044e-1, 1.4153185024193882e-3, -6.79231470631132637e-5, 6.14858667210896894e-6,
      -8.01655776235443082e-7, 1.32526289105552012e-7, -2.58930405315634027e-8, 5.72834344708168975e-9,
      -1.39537690343076657e-9, 3.67079831948957905e-10, -1.02678405759965503e-10, 3.02849074936736502e-11,
      -9.62765480622520539e-12, 3.12968527902585322e-12, -7.66521925899195137e-13, 2.38771056967415161e-13,
      -2.28763644588110236e-13, 8.77308336742980221e-14};
  constexpr double kP8[13] = {
      9.99457275788251954e-1, -5.36367319212967253e-4, 6.13741608010949751e-6, -2.05274482611706756e-7,
      1.28037614408009201e-8, -1.21210981789513772e-9, 1.55005654966325966e-10, -2.49114653547166607e-11,
      4.78699582136802789e-12, -1.01574850210656759e-12, 2.45317729673450063e-13, -1.02517900528310127e-13,
      3.33945225907080903e-14};
  constexpr double kQ8[16] = {
      -1.24440911036108149e-1, 5.46651927947510955e-4, -1.18171106612009754e-5, 5.68497188761874987e-7,
      -4.53497283736343393e-8, 5.14622526853905811e-9, -7.57633049889719997e-10, 1.36265138876174996e-10,
      -2.87072110711051457e-11, 6.87805487657686116e-12, -1.87364074354329584e-12, 5.57026680141996762e-13,
      -1.31375154988265364e-13, 3.75038522520632099e-14, -4.05740964240303386e-14, 1.71592236626347577e-14};
  const double PI = 3.14159265358979323846;
  if (x < 4.0) {
    const double s = fma(0.125 * x, x, -1.0);  // x^2 on [0, 16]
    const double J = horner(kJ0, s);
    *j0 = J;
    *y0 = fma((2.0 / PI) * log(0.5 * x), J, horner(kB0, s));
    return;
  }
  const double t = 1.0 / x, w = t * t;
  double P, Q;
  if (x < 8.0) {
    const double s = fma(128.0 / 3.0, w, -5.0 / 3.0);  // w on [1/64, 1/16]
    P = horner(kP4, s);
    Q = t * horner(kQ4, s);
  } else {
    const double s = fma(128.0, w, -1.0);  // w on [0, 1/64]
    P = horner(kP8, s);
    Q = t * horner(kQ8, s);
  }
  double s, c;
  sincos(x, &s, &c);
  const double a = sqrt(t * (1.0 / PI));  // sqrt(2/(pi x)) / sqrt 2, the cosine and sine of pi/4
  const double cp = c + s, sm = s - c;
  *j0 = a * (P * cp - Q * sm);
  *y0 = a * (P * sm + Q * cp);
}

// The same functions of a complex argument z (|arg z| < pi/2; the lossy 2D
// background has k r just above the real axis), by the same two methods with
// complex arithmetic: Hankel's expansion for |z| >= 25, Miller's backward
// recurrence with the same normalisation and Neumann's series (principal
// logarithm) below. Outputs are (re, im) pairs.
struct cz {
  double re, im;
};
__host__ __device__ inline cz czm(double a, double b) { return cz{a, b}; }
__host__ __device__ inline cz operator+(cz a, cz b) { return cz{a.re + b.re, a.im + b.im}; }
__host__ __device__ inline cz operator-(cz a, cz b) { return cz{a.re - b.re, a.im - b.im}; }
__host__ __device__ inline cz operator*(cz a, cz b) { return cz{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__host__ __device__ inline cz operator*(double s, cz a) { return cz{s * a.re, s * a.im}; }
__host__ __device__ inline cz czdiv(cz a, cz b) {
  // scaled division (Smith's method)
  if (fabs(b.re) >= fabs(b.im)) {
    const double r = b.im / b.re, d = b.re + r * b.im;
    return cz{(a.re + r * a.im) / d, (a.im - r * a.re) / d};
  }
  const double r = b.re / b.im, d = b.im + r * b.re;
  return cz{(r * a.re + a.im) / d, (r * a.im - a.re) / d};
}
__host__ __device__ inline double czabs(cz a) { return hypot(a.re, a.im); }
__host__ __device__ inline cz czsqrt(cz a) {
  const double m = czabs(a);
  const double re = sqrt(0.5 * (m + a.re)), im = sqrt(0.5 * (m - a.re));
  return cz{re, a.im < 0.0 ? -im : im};
}
__host__ __device__ inline cz czlog(cz a) { return cz{log(czabs(a)), atan2(a.im, a.re)}; }

__host__ __device__ inline void cbessel01(cz z, cz* j0, cz* j1, cz* y0, cz* y1) {
  const double PI = 3.14159265358979323846;
  const double EULER = 0.57721566490153286061;
  const double az = czabs(z);
  if (az >= 25.0) {
    const cz iz = czdiv(czm(1.0, 0.0), z);
    cz P0 = czm(1.0, 0.0), Q0 = czm(0.0, 0.0), P1 = czm(1.0, 0.0), Q1 = czm(0.0, 0.0);
    cz t0 = czm(1.0, 0.0), t1 = czm(1.0, 0.0);
    for (int k = 1; k <= 60; ++k) {
      const double f = (double)(2 * k - 1) * (double)(2 * k - 1);
      t0 = ((0.0 - f) / (8.0 * k)) * (t0 * iz);
      t1 = ((4.0 - f) / (8.0 * k)) * (t1 * iz);
      if (k & 1) {
        const double s = ((k - 1) / 2) & 1 ? -1.0 : 1.0;
        Q0 = Q0 + s * t0;
        Q1 = Q1 + s * t1;
      } else {
        const double s = (k / 2) & 1 ? -1.0 : 1.0;
        P0 = P0 + s * t0;
        P1 = P1 + s * t1;
      }
      if (czabs(t0) < 1e-18 && czabs(t1) < 1e-18) break;
    }
    // cos z, sin z of the complex argument
    double s, c;
    sincos(z.re, &s, &c);
    const double ch = cosh(z.im), sh = sinh(z.im);
    const cz cs = czm(c * ch, -s * sh), sn = czm(s * ch, c * sh);
    const double r2 = 0.70710678118654752440;
    const cz c0 = r2 * (cs + sn), s0 = r2 * (sn - cs);                  // chi = z - pi/4
    const cz c1 = r2 * (sn - cs), s1 = (-r2) * (sn + cs);               // chi = z - 3 pi/4
    const cz amp = czsqrt(czdiv(czm(2.0 / PI, 0.0), z));
    *j0 = amp * (P0 * c0 - Q0 * s0);
    *y0 = amp * (P0 * s0 + Q0 * c0);
    *j1 = amp * (P1 * c1 - Q1 * s1);
    *y1 = amp * (P1 * s1 + Q1 * c1);
    return;
  }
  const cz iz = czdiv(czm(1.0, 0.0), z);
  const int N = 2 * ((int)az + 20);
  cz fp = czm(0.0, 0.0), fc = czm(1.0, 0.0);
  cz S = czm(2.0, 0.0);
  cz sy0 = ((((N / 2) & 1) ? -1.0 : 1.0) / (N / 2)) * fc;
  cz sy1 = czm(0.0, 0.0), fodd = czm(0.0, 0.0), f1 = czm(0.0, 0.0);
  for (int k = N; k >= 1; --k) {
    const cz fm = (2.0 * k) * (iz * fc) - fp;
    fp = fc;
    fc = fm;
    const int m = k - 1;
    if (m & 1) {
      const int kk = (m + 1) / 2;
      sy1 = sy1 + (((kk & 1) ? -1.0 : 1.0) / kk) * (fc - fodd);
      fodd = fc;
      if (m == 1) f1 = fc;
    } else if (m >= 2) {
      S = S + 2.0 * fc;
      sy0 = sy0 + ((((m / 2) & 1) ? -1.0 : 1.0) / (m / 2)) * fc;
    } else {
      S = S + fc;
    }
    if (czabs(fc) > 1e250) {
      const double sc = 1e-250;
      fc = sc * fc; fp = sc * fp; fodd = sc * fodd; f1 = sc * f1; S = sc * S; sy0 = sc * sy0; sy1 = sc * sy1;
    }
  }
  const cz J0 = czdiv(fc, S), J1 = czdiv(f1, S);
  const cz lg = czlog(0.5 * z) + czm(EULER, 0.0);
  *j0 = J0;
  *j1 = J1;
  *y0 = (2.0 / PI) * (lg * J0) - (4.0 / PI) * czdiv(sy0, S);
  *y1 = (2.0 / PI) * (lg * J1 - J0 * iz) + (2.0 / PI) * czdiv(sy1, S);
}

// H0^(1)(z) = J0 + i Y0, the 2D Green's function's Hankel function, for a
// complex argument: for |z| >= 25 straight from Hankel's expansion,
// sqrt(2/(pi z)) (P0 + i Q0) e^{i (z - pi/4)} (no cancellation between J0 and
// Y0, which both grow like e^{Im z}; from |z| >= 15 when Im z >= 1); below
// from cbessel01.
__host__ __device__ inline cz chankel0(cz z) {
  const double PI = 3.14159265358979323846;
  const double az = czabs(z);
  // J0 + i Y0 loses e^{2 Im z} to cancellation: the expansion (error about
  // e^{-2|z|}) takes over from |z| = 15 once Im z >= 1
  if (az < 15.0 || (az < 25.0 && z.im < 1.0)) {
    cz j0, j1, y0, y1;
    cbessel01(z, &j0, &j1, &y0, &y1);
    return cz{j0.re - y0.im, j0.im + y0.re};
  }
  const cz iz = czdiv(czm(1.0, 0.0), z);
  cz P = czm(1.0, 0.0), Q = czm(0.0, 0.0), t = czm(1.0, 0.0);
  for (int k = 1; k <= 60; ++k) {
    const double f = (double)(2 * k - 1) * (double)(2 * k - 1);
    t = (-f / (8.0 * k)) * (t * iz);
    if (k & 1) Q = Q + ((((k - 1) / 2) & 1) ? -1.0 : 1.0) * t;
    else P = P + (((k / 2) & 1) ? -1.0 : 1.0) * t;
    if (czabs(t) < 1e-18) break;
  }
  double s, c;
  sincos(z.re - 0.25 * PI, &s, &c);
  const double d = exp(-z.im);
  const cz e = czm(d * c, d * s);
  const cz amp = czsqrt(czdiv(czm(2.0 / PI, 0.0), z));
  return amp * ((P + czm(-Q.im, Q.re)) * e);
}

}  // namespace fwi
