// Addressing of a pass tile whose pencils may cross signals: which pencil a
// tile's w-th one is and where its positions lie on either side.  Used by the mixed-radix and the chirp-z kernels.
#pragma once
#include "fft_common.hpp"

namespace lfft {
namespace dev {

// a table pointer read from the descriptor points to device memory
template <class T>
__device__ __forceinline__ const T* dev_ptr(const T* x) {
  return (const T*)(const __attribute__((address_space(1))) T*)x;
}

struct TileOf {
  long long b0;    // signal of the tile's first pencil
  int r0;          // its index o S + s inside the signal
  int n;           // pencils of this tile
};

struct Pencil {
  long long b;
  int o, s;
};

__device__ __forceinline__ Pencil pencil_of(const PassDesc& p, const TileOf& t, int w) {
  const unsigned r = (unsigned)(t.r0 + w);
  const unsigned q = fast_div(r, p.f_OS);
  const unsigned i = r - q * (unsigned)(p.O * p.S);
  Pencil c;
  c.b = t.b0 + q;
  c.o = (int)fast_div(i, p.f_S);
  c.s = (int)(i - (unsigned)c.o * (unsigned)p.S);
  return c;
}

__device__ __forceinline__ TileOf tile_of_pencils(const PassDesc& p, long long pen0, int width) {
  const long long OS = (long long)p.O * p.S, left = p.batch * OS - pen0;
  TileOf t;
  t.b0 = pen0 / OS;
  t.r0 = (int)(pen0 - t.b0 * OS);
  t.n = (int)(left < width ? left : width);
  return t;
}

// Element offsets (below 2^31) inside the signal of positions l0 + i step,
// i < R, of one pencil; the positions differ in one digit only.
template <int R, bool WIDE = false>
__device__ __forceinline__ void offsets(const PassDesc& p, const MapDesc& m, const Pencil& c, int l0,
                                        int step, unsigned* off) {
  if (m.mode == MAP_IDENTITY) {
    const unsigned a = ((unsigned)c.o * (unsigned)p.L + (unsigned)l0) * (unsigned)p.S + (unsigned)c.s;
#pragma unroll
    for (int i = 0; i < R; ++i) off[i] = a + (unsigned)(i * step) * (unsigned)p.S;
  } else if (m.mode == MAP_LINEAR) {
    const int4* Tl = dev_ptr(m.Tl);
    const unsigned a = (unsigned)(dev_ptr(m.To)[c.o].x + dev_ptr(m.Ts)[c.s].x) + (unsigned)Tl[l0].x;
    const unsigned d = R > 1 ? (unsigned)Tl[step].x : 0u;
#pragma unroll
    for (int i = 0; i < R; ++i) off[i] = a + (unsigned)i * d;
  } else {
    const int4 To = dev_ptr(m.To)[c.o], Ts = dev_ptr(m.Ts)[c.s], Tl = dev_ptr(m.Tl)[l0];
    const int4 D = R > 1 ? dev_ptr(m.Tl)[step] : make_int4(0, 0, 0, 0);
    if constexpr (WIDE) {
      // coordinates past 2^30: 64-bit sums
      long long x[4] = {0, 0, 0, 0};
      group_add(m, x, To);
      group_add(m, x, Ts);
      group_add(m, x, Tl);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        long long k = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) k += x[j] * m.box_stride[j];
        off[i] = (unsigned)k;
        if (i + 1 < R) group_add(m, x, D);
      }
    } else if (m.d == 2) {
      int c0 = To.x, c1 = To.y;
      gadd2(m, c0, c1, Ts);
      gadd2(m, c0, c1, Tl);
      const int h11 = m.H[1][1];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        off[i] = (unsigned)(c0 * h11 + c1);
        if (i + 1 < R) gadd2(m, c0, c1, D);
      }
    } else if (m.d == 3) {
      int x[4] = {To.x, To.y, To.z, 0};
      gadd3(m, x, Ts);
      gadd3(m, x, Tl);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        off[i] = (unsigned)nat_index3(m, x);
        if (i + 1 < R) gadd3(m, x, D);
      }
    } else {
      int x[4] = {To.x, To.y, To.z, To.w};
      gadd32(m, x, Ts);
      gadd32(m, x, Tl);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        off[i] = (unsigned)nat_index_i(m, x);
        if (i + 1 < R) gadd32(m, x, D);
      }
    }
  }
}

// position of l in the pencil's last digit
__device__ __forceinline__ unsigned post_pos(const PassDesc& p, unsigned l) {
  return l - fast_div(l, p.f_lmod) * (unsigned)p.post_lmod;
}

}  // namespace dev
}  // namespace lfft
