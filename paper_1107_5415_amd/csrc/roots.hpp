// Roots of unity at compile time, rounded to FP32, and what that rounding does
// to the length of a transformed vector.
#pragma once

namespace lfft {
namespace dev {

constexpr double kTwoPi = 6.283185307179586476925286766559;

// Taylor series on |x| <= pi/4
constexpr double sin_small(double x) {
  double t = x, s = x;
  for (int k = 1; k < 12; ++k) {
    t *= -x * x / ((2 * k) * (2 * k + 1));
    s += t;
  }
  return s;
}
constexpr double cos_small(double x) {
  double t = 1, s = 1;
  for (int k = 1; k < 12; ++k) {
    t *= -x * x / ((2 * k - 1) * (2 * k));
    s += t;
  }
  return s;
}
// cos and sin of 2 pi k / n, the angle reduced to an octant in integers
constexpr double cos_frac(int k, int n) {
  k %= n;
  if (2 * k > n) k = n - k;                     // [0, pi]
  if (4 * k > n) return -cos_frac(n - 2 * k, 2 * n);  // pi - x
  if (8 * k > n) return sin_small(kTwoPi * (n - 4 * k) / (4.0 * n));
  return cos_small(kTwoPi * k / n);
}
constexpr double sin_frac(int k, int n) {
  k %= n;
  if (2 * k > n) return -sin_frac(n - k, n);
  if (4 * k > n) return sin_frac(n - 2 * k, 2 * n);
  if (8 * k > n) return cos_small(kTwoPi * (n - 4 * k) / (4.0 * n));
  return sin_small(kTwoPi * k / n);
}

template <int N>
struct Roots {
  float c[N] = {}, s[N] = {};
  constexpr Roots() {
    for (int k = 0; k < N; ++k) {
      c[k] = (float)cos_frac(k, N);
      s[k] = (float)sin_frac(k, N);
    }
  }
};

// Gain of a register DFT of radix R: the mean of Re(conj(W) W') over its matrix
// W and the matrix W' that the rounded constants make.  They are the same in
// every butterfly, so what they add (up to 1.5e-8 a stage, 9e-8 in 10^6 points
// of radix 10) adds up.  The planner divides the output scale by it.
constexpr double root_gain(int k, int n) {
  return cos_frac(k, n) * (float)cos_frac(k, n) + sin_frac(k, n) * (float)sin_frac(k, n);
}
constexpr double rotations_gain(int A, int B) {   // the A x B rotations by (i j) / (A B)
  double g = 0;
  for (int i = 0; i < A; ++i)
    for (int j = 0; j < B; ++j) g += (i * j) % (A * B) ? root_gain(i * j, A * B) : 1.0;
  return g / (A * B);
}
inline double dft_gain(int R) {
  switch (R) {
    case 1: case 2: case 4: return 1.0;
    // even and odd inputs by half the radix, the odd ones' outputs rotated
    case 8: return rotations_gain(2, 4);
    case 16: return dft_gain(8) * rotations_gain(2, 8);
    case 6: return dft_gain(3);
    case 9: return dft_gain(3) * dft_gain(3) * rotations_gain(3, 3);
    case 10: return dft_gain(5);
    case 12: return dft_gain(3);
    case 14: return dft_gain(7);
    case 15: return dft_gain(3) * dft_gain(5);
    default: break;
  }
  // a prime: every root but 1 stands R - 1 times in the matrix
  double g = 2.0 * R - 1.0;
  for (int k = 1; k < R; ++k) g += (R - 1) * root_gain(k, R);
  return g / ((double)R * R);
}

}  // namespace dev
}  // namespace lfft
