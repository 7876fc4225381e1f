// In-register DFTs of any small length: odd primes by the symmetric sum over
// x_j + x_{p-j} and x_j - x_{p-j}, composites by two shorter ones.  The roots of unity are compile-time constants, evaluated in FP64 and
// rounded once.
#pragma once
#include "fft_common.hpp"
#include "roots.hpp"

namespace lfft {
namespace dev {

// f(k, X_k) for every output k of the DFT of odd length P, in pairs
// (k, P - k): with a = x_0 + sum_j cos(2 pi jk/P) (x_j + x_{P-j}) and
// b = sum_j sin(2 pi jk/P) (x_j - x_{P-j}), X_k = a + sign i b and
// X_{P-k} = a - sign i b.
template <int P, class F>
__device__ __forceinline__ void dft_odd_emit(const float2* v, int sign, F&& f) {
  constexpr Roots<P> w;
  constexpr int h = (P - 1) / 2;
  float2 s[h], d[h];
  float2 x0 = v[0];
#pragma unroll
  for (int j = 1; j <= h; ++j) {
    s[j - 1] = c_add(v[j], v[P - j]);
    d[j - 1] = c_sub(v[j], v[P - j]);
    x0 = c_add(x0, s[j - 1]);
  }
  const float2 y0 = v[0];
  f(0, x0);
#pragma unroll
  for (int k = 1; k <= h; ++k) {
    float2 a = y0, b = make_float2(0.f, 0.f);
#pragma unroll
    for (int j = 1; j <= h; ++j) {
      const float c = w.c[(j * k) % P], q = w.s[(j * k) % P];
      a.x += c * s[j - 1].x;
      a.y += c * s[j - 1].y;
      b.x += q * d[j - 1].x;
      b.y += q * d[j - 1].y;
    }
    b = c_muli(b, sign);
    f(k, c_add(a, b));
    f(P - k, c_sub(a, b));
  }
}

// v <- DFT of length R, exponent sign `sign`
template <int R>
__device__ __forceinline__ void dft_small(float2* v, int sign);

// R = A B: DFTs of length A over the inputs of step B, the twiddles
// exp(sign 2 pi i k1 i2 / R), then DFTs of length B; output k1 + A k2.
template <int A, int B>
__device__ __forceinline__ void dft_two(float2* v, int sign) {
  constexpr Roots<A * B> w;
  float2 t[B][A];
#pragma unroll
  for (int i2 = 0; i2 < B; ++i2) {
#pragma unroll
    for (int i1 = 0; i1 < A; ++i1) t[i2][i1] = v[B * i1 + i2];
    dft_small<A>(t[i2], sign);
#pragma unroll
    for (int k1 = 1; k1 < A; ++k1)
      if (i2 > 0) {
        const float c = w.c[(i2 * k1) % (A * B)], q = w.s[(i2 * k1) % (A * B)];
        t[i2][k1] = c_mul(t[i2][k1], make_float2(c, sign < 0 ? -q : q));
      }
  }
#pragma unroll
  for (int k1 = 0; k1 < A; ++k1) {
    float2 u[B];
#pragma unroll
    for (int i2 = 0; i2 < B; ++i2) u[i2] = t[i2][k1];
    dft_small<B>(u, sign);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = u[k2];
  }
}

// R = A B with A and B coprime: the inputs B n1 + A n2 and the outputs by their
// residues modulo A and B make it a plain A x B transform, without twiddles
// (Good's mapping), so with fewer products and roundings.
template <int A, int B>
__device__ __forceinline__ void dft_coprime(float2* v, int sign) {
  constexpr int R = A * B;
  float2 t[B][A];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) t[n2][n1] = v[(B * n1 + A * n2) % R];
    dft_small<A>(t[n2], sign);
  }
#pragma unroll
  for (int k1 = 0; k1 < A; ++k1) {
    float2 u[B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) u[n2] = t[n2][k1];
    dft_small<B>(u, sign);
#pragma unroll
    for (int k = k1; k < R; k += A) v[k] = u[k % B];
  }
}

template <int R>
__device__ __forceinline__ void dft_small(float2* v, int sign) {
  if constexpr ((R & (R - 1)) == 0) {
    dft_pow2<R>(v, sign);
  } else if constexpr (R == 3) {
    dft3(v, sign);
  } else if constexpr (R == 6) {
    dft_coprime<2, 3>(v, sign);
  } else if constexpr (R == 9) {
    dft_two<3, 3>(v, sign);
  } else if constexpr (R == 10) {
    dft_coprime<2, 5>(v, sign);
  } else if constexpr (R == 12) {
    dft_coprime<4, 3>(v, sign);
  } else if constexpr (R == 14) {
    dft_coprime<2, 7>(v, sign);
  } else if constexpr (R == 15) {
    dft_coprime<3, 5>(v, sign);
  } else {
    float2 y[R];
    dft_odd_emit<R>(v, sign, [&](int k, float2 x) { y[k] = x; });
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = y[k];
  }
}

}  // namespace dev
}  // namespace lfft
