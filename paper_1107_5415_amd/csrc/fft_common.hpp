// Device helpers shared by the FFT pass kernels: complex arithmetic,
// in-register DFTs of small lengths and the natural-order group arithmetic
// of the gather/scatter maps.
#pragma once
#include <hip/hip_runtime.h>

#include "device.hpp"

namespace lfft {
namespace dev {

__device__ __forceinline__ float2 c_mul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 c_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 c_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 c_conj(float2 a) { return make_float2(a.x, -a.y); }
// a * (sign * i)
__device__ __forceinline__ float2 c_muli(float2 a, int sign) {
  return sign < 0 ? make_float2(a.y, -a.x) : make_float2(-a.y, a.x);
}
// a (s + lo)
__device__ __forceinline__ float2 c_scale(float2 a, float s, float lo) {
  return make_float2(fmaf(a.x, s, a.x * lo), fmaf(a.y, s, a.y * lo));
}
__device__ __forceinline__ float2 tw_lookup(const float2* tw, long long k, int sign) {
  float2 w = tw[k];
  return sign < 0 ? w : c_conj(w);
}

// In-register DFT of power-of-two length R with exponent sign `sign`.
template <int R>
__device__ __forceinline__ void dft_pow2(float2* v, int sign);

template <>
__device__ __forceinline__ void dft_pow2<1>(float2*, int) {}

template <>
__device__ __forceinline__ void dft_pow2<2>(float2* v, int) {
  float2 a = v[0], b = v[1];
  v[0] = c_add(a, b);
  v[1] = c_sub(a, b);
}

template <>
__device__ __forceinline__ void dft_pow2<4>(float2* v, int sign) {
  float2 s02 = c_add(v[0], v[2]), d02 = c_sub(v[0], v[2]);
  float2 s13 = c_add(v[1], v[3]), d13 = c_muli(c_sub(v[1], v[3]), sign);
  v[0] = c_add(s02, s13);
  v[2] = c_sub(s02, s13);
  v[1] = c_add(d02, d13);
  v[3] = c_sub(d02, d13);
}

// exp(sign * 2 pi i k / 16) for k in [0, 8): cos and sin of multiples of pi/8
__device__ __forceinline__ float2 root16(int k, int sign) {
  constexpr float C[8] = {1.0f, 0.92387953251128675613f, 0.70710678118654752440f,
                          0.38268343236508977173f, 0.0f, -0.38268343236508977173f,
                          -0.70710678118654752440f, -0.92387953251128675613f};
  constexpr float Sn[8] = {0.0f, 0.38268343236508977173f, 0.70710678118654752440f,
                           0.92387953251128675613f, 1.0f, 0.92387953251128675613f,
                           0.70710678118654752440f, 0.38268343236508977173f};
  return make_float2(C[k], sign < 0 ? -Sn[k] : Sn[k]);
}

// o * exp(sign 2 pi i K / R) for a compile-time K < R / 2: the factors 1
// and sign * i cost no multiplication (IEEE semantics keep the compiler
// from dropping products with the constant 0 by itself).
template <int R, int K>
__device__ __forceinline__ float2 rot_k(float2 o, int sign) {
  if constexpr (K == 0) {
    return o;
  } else if constexpr (4 * K == R) {
    return c_muli(o, sign);
  } else {
    return c_mul(root16(K * (16 / R), sign), o);
  }
}

// butterflies k = K .. R/2 - 1 of the last combining step
template <int R, int K>
struct Combine {
  __device__ __forceinline__ static void run(float2* v, const float2* e, const float2* o, int sign) {
    if constexpr (K < R / 2) {
      const float2 t = rot_k<R, K>(o[K], sign);
      v[K] = c_add(e[K], t);
      v[K + R / 2] = c_sub(e[K], t);
      Combine<R, K + 1>::run(v, e, o, sign);
    }
  }
};

template <int R>
__device__ __forceinline__ void dft_pow2(float2* v, int sign) {
  static_assert(R <= 16, "radix above 16");
  // even/odd split: X[k] = E[k] + w^k O[k], X[k + R/2] = E[k] - w^k O[k]
  float2 e[R / 2], o[R / 2];
#pragma unroll
  for (int i = 0; i < R / 2; ++i) {
    e[i] = v[2 * i];
    o[i] = v[2 * i + 1];
  }
  dft_pow2<R / 2>(e, sign);
  dft_pow2<R / 2>(o, sign);
  Combine<R, 0>::run(v, e, o, sign);
}

// Twiddles of a butterfly of radix R <= 16: input i is multiplied by w^i.
// The powers 1 .. 3, 4, 8 and 12 (those below R) come from the table, the
// others are one product of two of them (from w, w^2, w^4 and w^8 alone they
// would be up to three in a row).
constexpr int tw_bases(int R) { return R <= 4 ? R - 1 : R <= 8 ? 4 : R <= 12 ? 5 : 6; }
constexpr int tw_exponent(int k) { return k < 4 ? k + 1 : 4 * (k - 2); }

template <int R, int I = 1>
__device__ __forceinline__ void apply_twiddles(float2* x, const float2* b) {
  if constexpr (I < R) {
    constexpr int lo = I & 3, hi = I >> 2;
    if constexpr (hi == 0)
      x[I] = c_mul(x[I], b[lo - 1]);
    else if constexpr (lo == 0)
      x[I] = c_mul(x[I], b[hi + 2]);
    else
      x[I] = c_mul(x[I], c_mul(b[hi + 2], b[lo - 1]));
    apply_twiddles<R, I + 1>(x, b);
  }
}

// v[i] <- v[(i - k) mod R], 0 <= k < R, different in every lane: a select per
// value and bit of k, and no rounding.  In place, one cycle after the other.
template <int R, int S = 1>
__device__ __forceinline__ void rotate_by(float2* v, int k) {
  if constexpr (S < R) {
    const bool on = (k & S) != 0;
#pragma unroll
    for (int r = 0; r < S; ++r) {
      const float2 last = v[R - S + r];
#pragma unroll
      for (int i = R - S + r; i >= S; i -= S) {
        v[i].x = on ? v[i - S].x : v[i].x;
        v[i].y = on ? v[i - S].y : v[i].y;
      }
      v[r].x = on ? last.x : v[r].x;
      v[r].y = on ? last.y : v[r].y;
    }
    rotate_by<R, 2 * S>(v, k);
  }
}

__device__ __forceinline__ void dft3(float2* v, int sign) {
  const float h = 0.86602540378443864676f;  // sqrt(3)/2
  float2 t1 = c_add(v[1], v[2]);
  float2 t2 = c_sub(v[1], v[2]);
  float2 x0 = v[0];
  v[0] = c_add(x0, t1);
  float2 mm = make_float2(x0.x - 0.5f * t1.x, x0.y - 0.5f * t1.y);
  float2 nn = c_muli(make_float2(h * t2.x, h * t2.y), sign);
  v[1] = c_add(mm, nn);
  v[2] = c_sub(mm, nn);
}

// c += b in Z^d / H Z^d for reduced c and b in 64 bits (lattices of 2^30
// points and more): coordinate i needs at most 4 - i subtractions of column i
// and 3 - i additions, as in gadd32 below.  Unrolled so that c stays in
// registers; the columns beyond d are never used.
__device__ __forceinline__ void group_add(const MapDesc& m, long long* c, int4 b) {
  c[0] += b.x;
  c[1] += b.y;
  c[2] += b.z;
  c[3] += b.w;
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    if (i < m.d) {
#pragma unroll
      for (int t = 0; t < 4 - i; ++t) {
        const bool over = c[i] >= m.H[i][i];
#pragma unroll
        for (int r = 0; r <= i; ++r) c[r] -= over ? m.H[r][i] : 0;
      }
#pragma unroll
      for (int t = 0; t < 3 - i; ++t) {
        const bool under = c[i] < 0;
#pragma unroll
        for (int r = 0; r <= i; ++r) c[r] += under ? m.H[r][i] : 0;
      }
    }
  }
}

}  // namespace dev
}  // namespace lfft

namespace lfft {
namespace dev {

// Group sum in Z^d / H Z^d of two reduced coordinate vectors (int32; the
// planner routes lattices with m >= 2^30 to the mixed-radix kernel).
__device__ __forceinline__ void gadd32(const MapDesc& m, int* c, int4 b) {
  c[0] += b.x;
  c[1] += b.y;
  c[2] += b.z;
  c[3] += b.w;
  // Both operands are reduced.  Processing coordinates from the last one,
  // coordinate i has received at most k = d - 1 - i corrections of size
  // below H_ii from the later columns, so it lies in (-k H_ii, (2 + k) H_ii)
  // and needs at most k + 1 subtractions or k additions of column i.
  // Branch-free selects, fully unrolled so that c stays in registers.
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    if (i < m.d) {
      const int k = m.d - 1 - i;
#pragma unroll
      for (int t = 0; t < 4 - i; ++t) {
        if (t <= k) {
          const bool over = c[i] >= m.H[i][i];
#pragma unroll
          for (int r = 0; r <= i; ++r) c[r] -= over ? m.H[r][i] : 0;
        }
      }
#pragma unroll
      for (int t = 0; t < 3 - i; ++t) {
        if (t < k) {
          const bool under = c[i] < 0;
#pragma unroll
          for (int r = 0; r <= i; ++r) c[r] += under ? m.H[r][i] : 0;
        }
      }
    }
  }
}

// four-step twiddle exp(sign 2 pi i k lo / postN): k < post_lmod and
// lo < lo_n, so the product stays below postN = post_lmod lo_n
__device__ __forceinline__ float2 post_twiddle(const PassDesc& p, unsigned x) {
  float2 w = c_mul(p.tw_hi[x >> 12], p.tw_lo[x & 4095]);
  if (p.sign > 0) w.y = -w.y;
  return w;
}

__device__ __forceinline__ unsigned post_lo(const PassDesc& p, int s) {
  const unsigned q = fast_div((unsigned)s, p.f_lodiv);
  return q - fast_div(q, p.f_lon) * (unsigned)p.lo_n;
}

// Workgroups are dispatched round-robin over the 8 XCDs of the MI355X.  Map
// dispatch index i to a logical tile so that every XCD works on one
// contiguous range of tiles: concurrently running neighbours share cache
// lines in that XCD's L2 (partial-line reads hit, partial-line writes merge).
__device__ __forceinline__ long long xcd_tile(long long i, long long n) {
  const long long per = n >> 3, rem = n & 7;
  const long long x = i & 7, k = i >> 3;
  return x * per + (x < rem ? x : rem) + k;
}

// Touch every 64-byte line of the kernel's first BYTES bytes of arguments at
// once.  The pass descriptor spans two dozen lines outside the device's own
// memory; read where they are needed, one dependent step after the other, each
// new line adds its latency to every wave.
template <int BYTES>
__device__ __forceinline__ void touch_args() {
  typedef const __attribute__((address_space(4))) int* Arg;
  const Arg k = (Arg)__builtin_amdgcn_kernarg_segment_ptr();
  int acc = 0;
#pragma unroll
  for (int i = 0; i < (BYTES + 63) / 64; ++i) acc |= k[16 * i];
  asm volatile("" ::"s"(acc));
}

// The kernel's first argument in place.  A by-value descriptor whose input and
// output maps meet in one address (kernels with both sides natural) would be
// copied to scratch memory, 1.4 KB per thread.
template <class T>
__device__ __forceinline__ const T& first_arg() {
  typedef const __attribute__((address_space(4))) T* Arg;
  return *(const T*)(Arg)__builtin_amdgcn_kernarg_segment_ptr();
}

// Non-temporal 8-byte load and store: the line is not kept for reuse.  For
// data read or written once by a call (whole lines, so that no other wave
// has to fetch the same line again), which leaves the caches to the data
// that is read again.
typedef float stream_f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 load_stream(const float2* p) {
  const stream_f2 t = __builtin_nontemporal_load(reinterpret_cast<const stream_f2*>(p));
  return make_float2(t.x, t.y);
}
__device__ __forceinline__ void store_stream(float2* p, float2 v) {
  const stream_f2 t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<stream_f2*>(p));
}

// Natural box of a 2-D lattice, column Hermite form [[h00, h01], [0, h11]]:
// c += b for reduced c and b.  c1 + b1 < 2 h11 needs at most one column-1
// subtraction; c0 then lies in (-h00, 2 h00 - 1) and needs at most one
// correction by h00.
__device__ __forceinline__ void gadd2(const MapDesc& m, int& c0, int& c1, int4 b) {
  c0 += b.x;
  c1 += b.y;
  const bool o1 = c1 >= m.H[1][1];
  c1 -= o1 ? m.H[1][1] : 0;
  c0 -= o1 ? m.H[0][1] : 0;
  c0 += c0 < 0 ? m.H[0][0] : 0;
  c0 -= c0 >= m.H[0][0] ? m.H[0][0] : 0;
}

// Natural box of a 3-D lattice (upper-triangular H): c += b for reduced c
// and b.  Coordinate 2 needs at most one subtraction of column 2, which
// leaves coordinate 1 in (-h11, 2 h11 - 1): one correction by column 1;
// coordinate 0 then lies in (-2 h00, 3 h00 - 2): at most two corrections.
__device__ __forceinline__ void gadd3(const MapDesc& m, int* c, int4 b) {
  c[0] += b.x;
  c[1] += b.y;
  c[2] += b.z;
  const bool o2 = c[2] >= m.H[2][2];
  c[2] -= o2 ? m.H[2][2] : 0;
  c[1] -= o2 ? m.H[1][2] : 0;
  c[0] -= o2 ? m.H[0][2] : 0;
  const bool u1 = c[1] < 0, o1 = c[1] >= m.H[1][1];
  c[1] += u1 ? m.H[1][1] : (o1 ? -m.H[1][1] : 0);
  c[0] += u1 ? m.H[0][1] : (o1 ? -m.H[0][1] : 0);
  const int h00 = m.H[0][0];
  c[0] += c[0] < 0 ? h00 : 0;
  c[0] += c[0] < 0 ? h00 : 0;
  c[0] -= c[0] >= h00 ? h00 : 0;
  c[0] -= c[0] >= h00 ? h00 : 0;
}

__device__ __forceinline__ int nat_index3(const MapDesc& m, const int* c) {
  return c[0] * (int)m.box_stride[0] + c[1] * (int)m.box_stride[1] + c[2];
}

// linear natural index (int: the planner keeps these lattices below 2^30 points)
__device__ __forceinline__ int nat_index_i(const MapDesc& m, const int* c) {
  int idx = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < m.d) idx += c[i] * (int)m.box_stride[i];
  return idx;
}

__device__ __forceinline__ long long nat_index32(const MapDesc& m, const int* c) {
  long long idx = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < m.d) idx += (long long)c[i] * m.box_stride[i];
  return idx;
}

}  // namespace dev
}  // namespace lfft
