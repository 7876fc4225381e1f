// Chirp-z (Bluestein) passes: the DFT of one grid axis, or of one four-step
// digit of an axis, whose length L has a prime factor too large for a register
// butterfly (a few such digits are direct sums, see the planner).  With w = exp(-2 pi i / L) and
// jk = (j^2 + k^2 - (k - j)^2) / 2,
//   X_k = sum_j x_j w^{jk} = c_k sum_j (x_j c_j) conj(c_{k-j}),  c_j = w^{j^2/2},
// a cyclic convolution of length N >= 2L - 1 (a power of two).  The axis is
// one factor of the Kronecker form of the lattice Fourier matrix (Section 4.1,
// Theorem 1), so Algorithm 1 of Section 4.2 applies to any elementary
// divisors.
//
// The convolution never leaves the chip between its two FFTs: with the radix
// sequence of the second FFT the reverse of the first one's, the values a
// thread holds after the last stage of the first FFT are the ones it needs
// for the first stage of the second, so multiplying by the kernel's DFT costs
// no exchange.
//  * L <= 8192 (N <= 16384): one launch.  Load (gather and chirp), FFT,
//    product, inverse FFT, store (chirp and scatter), W pencils per workgroup
//    and 16 values per thread.
//  * longer axes: three launches over a workspace of N points per pencil,
//    N = H R with element n = a R + c: columns (gather, chirp, FFT over a,
//    twiddle W_N^{bc}), rows in place (FFT over c, product, inverse FFT,
//    conjugate twiddle), columns (inverse FFT over b, chirp, scatter).
// Bound by latency at the sizes of arbitrary integer matrices (10^4 .. 10^5
// points, a few dozen to a few hundred workgroups), so what counts is the
// number of launches and of LDS round trips in each: 2 x 69512 points forward
// and back (prime 8689) took 193 us as seven launches per transform (gather,
// two FFTs of two passes, product, scatter), 47 us as three.
#include <hip/hip_runtime.h>

#include <atomic>

#include "chirp.hpp"
#include "fft_common.hpp"
#include "kernels.hpp"
#include "ktrace.hpp"
#include "pass_addr.hpp"

namespace lfft {
namespace {
using namespace dev;

constexpr int kV = 16;   // values per thread

// Radix of stage s of an N-point transform: 16 first (no twiddles).
__host__ __device__ constexpr int radix_at(int N, int s) {
  return N == 16384 ? (s < 2 ? 16 : 8)
       : N == 8192  ? (s < 1 ? 16 : 8)
       : N == 4096  ? 16
       : N == 2048  ? (s < 2 ? 16 : 8)
       : N == 1024  ? (s < 1 ? 16 : 8)
       : N == 512   ? (s < 1 ? 16 : s < 2 ? 8 : 4)
       : N == 256   ? 16
       : (s < 1 ? 16 : 8);   // 128
}
__host__ __device__ constexpr int stages(int N) {
  return N >= 8192 ? 4 : N >= 512 ? 3 : 2;
}
// the second FFT of a convolution runs the radices backwards
template <int N, bool REV>
struct Seq {
  static constexpr int n = stages(N);
  static constexpr int r(int s) { return radix_at(N, REV ? n - 1 - s : s); }
  static constexpr int ns(int s) { return s == 0 ? 1 : ns(s - 1) * r(s - 1); }
};

__device__ __forceinline__ int phys(int e) { return e + (e >> 4); }

// LDS position of pencil position l of tile pencil w
template <int N, int W, bool ACROSS>
__device__ __forceinline__ int at(int l, int w) {
  return phys(ACROSS ? l * W + w : w * N + l);
}

// w^i, i = 1 .. R - 1, from w^(2^k), the exponents below N
template <int R, int I>
__device__ __forceinline__ void powers(float2* v, float2* pw) {
  if constexpr (I < R) {
    constexpr int hb = chirp_high_bit(I);
    if constexpr (hb != I) pw[I] = c_mul(pw[hb], pw[I - hb]);
    v[I] = c_mul(v[I], pw[I]);
    powers<R, I + 1>(v, pw);
  }
}

// Stages SI .. of the transform of the kV values a thread holds in the order
// of stage SI's inputs (butterfly q, input i at value q R + i: position
// jt + T q + i N / R with T threads per pencil).  Returns with the outputs of
// the last stage, at positions jt + T q + i N / R too.  tw[k] =
// exp(-2 pi i k / N).
template <int N, int W, bool ACROSS, bool REV, int SI>
__device__ __forceinline__ void transform(float2* v, float2* lds, const float2* __restrict__ tw,
                                          int jt, int w, int sign) {
  using S = Seq<N, REV>;
  constexpr int R = S::r(SI), Ns = S::ns(SI), T = N / kV;
#pragma unroll
  for (int q = 0; q < kV / R; ++q) {
    float2* x = v + q * R;
    if constexpr (SI > 0) {
      const int e = ((jt + T * q) & (Ns - 1)) * (N / (Ns * R));
      float2 pw[R];
#pragma unroll
      for (int i = 1; i < R; i *= 2) {
        pw[i] = tw[e * i];
        if (sign > 0) pw[i].y = -pw[i].y;
      }
      powers<R, 1>(x, pw);
    }
    dft_pow2<R>(x, sign);
  }
  if constexpr (SI + 1 < S::n) {
    constexpr int R2 = S::r(SI + 1);
#pragma unroll
    for (int q = 0; q < kV / R; ++q) {
      const int j = jt + T * q;
      const int o = (j / Ns) * (Ns * R) + (j & (Ns - 1));
#pragma unroll
      for (int i = 0; i < R; ++i) lds[at<N, W, ACROSS>(o + i * Ns, w)] = v[q * R + i];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kV / R2; ++q)
#pragma unroll
      for (int i = 0; i < R2; ++i)
        v[q * R2 + i] = lds[at<N, W, ACROSS>(jt + T * q + i * (N / R2), w)];
    __syncthreads();
    transform<N, W, ACROSS, REV, SI + 1>(v, lds, tw, jt, w, sign);
  }
}

// v <- inverse FFT(FFT(v) . bhat), unnormalised (1 / N is in bhat); in and
// out: value i at position jt + i N / 16.
template <int N, int W, bool ACROSS>
__device__ __forceinline__ void convolve(float2* v, float2* lds, const float2* __restrict__ tw,
                                         const float2* __restrict__ bhat, int jt, int w, int sign) {
  constexpr int R = Seq<N, true>::r(0), T = N / kV;
  transform<N, W, ACROSS, false, 0>(v, lds, tw, jt, w, -1);
#pragma unroll
  for (int q = 0; q < kV / R; ++q)
#pragma unroll
    for (int i = 0; i < R; ++i) {
      float2 h = bhat[jt + T * q + i * (N / R)];
      if (sign > 0) h.y = -h.y;
      v[q * R + i] = c_mul(v[q * R + i], h);
    }
  transform<N, W, ACROSS, true, 0>(v, lds, tw, jt, w, 1);
}

__device__ __forceinline__ float2 chirp_at(const PassDesc& p, int j) {
  float2 c = p.chirp[j];
  return p.sign < 0 ? c : c_conj(c);
}

// threads of a tile: across the W pencils first, or along one
template <int W, bool ACROSS, int T>
__device__ __forceinline__ void lane_of(int& w, int& jt) {
  const int tid = threadIdx.x;
  w = ACROSS ? tid % W : tid / T;
  jt = ACROSS ? tid / W : tid % T;
}

__device__ __forceinline__ TileOf chirp_tile(const PassDesc& p, int W, long long block, long long n) {
  return tile_of_pencils(p, xcd_tile(block, n) * W, W);
}

template <int N, int W, bool ACROSS>
__global__ void __launch_bounds__(W* N / kV)
    chirp_tile_kernel(PassDesc p, const float2* __restrict__ in, float2* __restrict__ out) {
  extern __shared__ float2 lds[];
  constexpr int T = N / kV;
  int w, jt;
  lane_of<W, ACROSS, T>(w, jt);
  const TileOf t = chirp_tile(p, W, blockIdx.x, gridDim.x);
  const bool active = w < t.n;
  const Pencil pc = pencil_of(p, t, active ? w : 0);
  float2 v[kV];
  {
    unsigned off[kV];
    offsets<kV>(p, p.in, pc, jt, T, off);
    const float2* src = in + pc.b * p.in.bstride;
#pragma unroll
    for (int i = 0; i < kV; ++i) {
      const int l = jt + i * T;
      v[i] = make_float2(0.f, 0.f);
      if (active && l < p.L) v[i] = c_mul(src[off[i]], chirp_at(p, l));
    }
  }
  convolve<N, W, ACROSS>(v, lds, p.tw_row, p.bhat, jt, w, p.sign);
  if (active) {
    unsigned off[kV];
    offsets<kV>(p, p.out, pc, jt, T, off);
    float2* dst = out + pc.b * p.out.bstride;
    const unsigned lo = p.post ? post_lo(p, pc.s) : 0u;
#pragma unroll
    for (int i = 0; i < kV; ++i) {
      const int l = jt + i * T;
      if (l >= p.L) continue;
      float2 x = c_mul(v[i], chirp_at(p, l));
      if (p.post) x = c_mul(x, post_twiddle(p, (unsigned)l * lo));
      dst[off[i]] = c_scale(x, p.scale, p.scale_lo);
    }
  }
}

// W_N^x conjugated for conj = true, N = p.bN
__device__ __forceinline__ float2 conv_twiddle(const PassDesc& p, int x, bool conj) {
  float2 t = c_mul(p.cv_hi[x >> 12], p.cv_lo[x & 4095]);
  if (conj) t.y = -t.y;
  return t;
}

// Columns of a long axis: one workgroup takes W neighbouring columns c of one
// pencil (WIDE: 64-bit coordinates).  IN: gather and chirp, FFT over a, twiddle, to A; otherwise from A,
// inverse FFT over b, chirp and scatter.
template <int H, int W, bool IN, bool WIDE>
__global__ void __launch_bounds__(W* H / kV)
    chirp_cols_kernel(PassDesc p, const float2* __restrict__ in, float2* __restrict__ out) {
  extern __shared__ float2 lds[];
  constexpr int T = H / kV;
  const int w = threadIdx.x % W, jt = threadIdx.x / W;
  const int Rw = p.bN / H;                 // columns of one pencil, a multiple of W
  const long long tile = xcd_tile(blockIdx.x, gridDim.x);
  const int per = Rw / W;
  const long long pen = tile / per;
  const int c = (int)(tile - pen * per) * W + w;
  const TileOf t = tile_of_pencils(p, pen, 1);
  const Pencil pc = pencil_of(p, t, 0);
  float2 v[kV];
  unsigned off[kV];
  const MapDesc& m = IN ? p.in : p.out;
  // positions l = c + a R, a = jt + i T; c < R < L and T R < L, so both are
  // entries of the map's table
  const int l0 = c + jt * Rw;
  const bool some = l0 < p.L;
  offsets<kV, WIDE>(p, m, pc, some ? l0 : c, T * Rw, off);
  if constexpr (IN) {
    const float2* src = in + pc.b * m.bstride;
#pragma unroll
    for (int i = 0; i < kV; ++i) {
      const long long l = l0 + (long long)i * T * Rw;
      v[i] = make_float2(0.f, 0.f);
      if (l < p.L) v[i] = c_mul(src[off[i]], chirp_at(p, (int)l));
    }
    transform<H, W, true, false, 0>(v, lds, p.tw_col, jt, w, -1);
    constexpr int R = Seq<H, true>::r(0);
    float2* A = out + pen * p.bN;
#pragma unroll
    for (int q = 0; q < kV / R; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int b = jt + T * q + i * (H / R);
        A[b * Rw + c] = c_mul(v[q * R + i], conv_twiddle(p, b * c, false));
      }
  } else {
    constexpr int R = Seq<H, true>::r(0);
    const float2* A = in + pen * p.bN;
#pragma unroll
    for (int q = 0; q < kV / R; ++q)
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int b = jt + T * q + i * (H / R);
        v[q * R + i] = A[b * Rw + c];
      }
    transform<H, W, true, true, 0>(v, lds, p.tw_col, jt, w, 1);
    float2* dst = out + pc.b * m.bstride;
#pragma unroll
    for (int i = 0; i < kV; ++i) {
      const long long l = l0 + (long long)i * T * Rw;
      if (l >= p.L) continue;
      const float2 x = c_mul(v[i], chirp_at(p, (int)l));
      dst[off[i]] = c_scale(x, p.scale, p.scale_lo);
    }
  }
}

// Rows of a long axis, in place: row b of a pencil times its part of the
// kernel's DFT (table in the same (b, e) order), and the twiddle of the
// inverse transform.
template <int N, int W>
__global__ void __launch_bounds__(W* N / kV) chirp_rows_kernel(PassDesc p, float2* __restrict__ A) {
  extern __shared__ float2 lds[];
  constexpr int T = N / kV;
  int w, jt;
  lane_of<W, false, T>(w, jt);
  const int H = p.bN / N;                  // rows of one pencil, a multiple of W
  const long long row = xcd_tile(blockIdx.x, gridDim.x) * W + w;
  const int b = (int)(row % H);
  float2* x = A + row * N;
  float2 v[kV];
#pragma unroll
  for (int i = 0; i < kV; ++i) v[i] = x[jt + i * T];
  convolve<N, W, false>(v, lds, p.tw_row, p.bhat + (long long)b * N, jt, w, p.sign);
#pragma unroll
  for (int i = 0; i < kV; ++i) {
    const int c = jt + i * T;
    x[c] = c_mul(v[i], conv_twiddle(p, b * c, true));
  }
}

constexpr size_t lds_of(int elems) { return (size_t)(elems + elems / 16 + 1) * sizeof(float2); }

// allow the largest tile's LDS once per kernel; threads that race here all
// write the same attribute
template <class K>
hipError_t allow_lds(K k, std::atomic<bool>& done, size_t lds) {
  if (done.load(std::memory_order_acquire)) return hipSuccess;
  hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e == hipSuccess) done.store(true, std::memory_order_release);
  return e;
}

template <int N, bool ACROSS>
hipError_t launch_tile(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  constexpr int W = chirp_width(N);
  static std::atomic<bool> ok{false};
  hipError_t e = allow_lds(chirp_tile_kernel<N, W, ACROSS>, ok, lds_of(W * N));
  if (e != hipSuccess) return e;
  const long long npen = p.batch * (long long)p.O * p.S, tiles = (npen + W - 1) / W;
  if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((chirp_tile_kernel<N, W, ACROSS>), dim3((unsigned)tiles), dim3(W * N / kV),
                     lds_of(W * N), s, p, in, out);
  return hipGetLastError();
}

template <int N>
hipError_t launch_tile_n(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  if constexpr (chirp_width(N) > 1)
    if (p.out.across) return launch_tile<N, true>(p, in, out, s);
  return launch_tile<N, false>(p, in, out, s);
}

template <int H, bool IN, bool WIDE>
hipError_t launch_cols(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  constexpr int W = chirp_col_width(H);
  static std::atomic<bool> ok{false};
  hipError_t e = allow_lds(chirp_cols_kernel<H, W, IN, WIDE>, ok, lds_of(W * H));
  if (e != hipSuccess) return e;
  const long long tiles = p.batch * (long long)p.O * p.S * (p.bN / H / W);
  if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((chirp_cols_kernel<H, W, IN, WIDE>), dim3((unsigned)tiles), dim3(W * H / kV),
                     lds_of(W * H), s, p, in, out);
  return hipGetLastError();
}

template <int N>
hipError_t launch_rows(const PassDesc& p, float2* A, hipStream_t s) {
  constexpr int W = chirp_width(N);
  static std::atomic<bool> ok{false};
  hipError_t e = allow_lds(chirp_rows_kernel<N, W>, ok, lds_of(W * N));
  if (e != hipSuccess) return e;
  const long long tiles = p.batch * (long long)p.O * p.S * (p.bN / N) / W;
  if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((chirp_rows_kernel<N, W>), dim3((unsigned)tiles), dim3(W * N / kV),
                     lds_of(W * N), s, p, A);
  return hipGetLastError();
}

template <bool IN, bool WIDE>
hipError_t launch_cols_h(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  if (p.bN < 2 * p.L - 1 || p.bH < 1 || p.bN % p.bH != 0 || p.bN / p.bH < 256)
    return hipErrorInvalidValue;
  switch (p.bH) {
    case 128: return launch_cols<128, IN, WIDE>(p, in, out, s);
    case 256: return launch_cols<256, IN, WIDE>(p, in, out, s);
    case 512: return launch_cols<512, IN, WIDE>(p, in, out, s);
    case 1024: return launch_cols<1024, IN, WIDE>(p, in, out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

std::vector<int> chirp_radices(int N, bool second) {
  std::vector<int> r;
  for (int i = 0; i < stages(N); ++i) r.push_back(radix_at(N, second ? stages(N) - 1 - i : i));
  return r;
}

const char* chirp_kernel_name(const PassDesc& p, int step) {
  if (p.kind == 5)
    return kernel_name_intern("chirp_tile_kernel<%d, %d, %s>", p.bN, chirp_width(p.bN),
                              p.out.across && chirp_width(p.bN) > 1 ? "true" : "false");
  if (step == 1)
    return kernel_name_intern("chirp_rows_kernel<%d, %d>", p.bN / p.bH, chirp_width(p.bN / p.bH));
  return kernel_name_intern("chirp_cols_kernel<%d, %d, %s, %s>", p.bH, chirp_col_width(p.bH),
                            step == 0 ? "true" : "false", p.wide ? "true" : "false");
}

hipError_t launch_chirp_tile(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  if (p.bN < 2 * p.L - 1) return hipErrorInvalidValue;
  switch (p.bN) {
    case 128: return launch_tile_n<128>(p, in, out, s);
    case 256: return launch_tile_n<256>(p, in, out, s);
    case 512: return launch_tile_n<512>(p, in, out, s);
    case 1024: return launch_tile_n<1024>(p, in, out, s);
    case 2048: return launch_tile_n<2048>(p, in, out, s);
    case 4096: return launch_tile_n<4096>(p, in, out, s);
    case 8192: return launch_tile_n<8192>(p, in, out, s);
    case 16384: return launch_tile_n<16384>(p, in, out, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_chirp_in(const PassDesc& p, const float2* in, float2* A, hipStream_t s) {
  return p.wide ? launch_cols_h<true, true>(p, in, A, s) : launch_cols_h<true, false>(p, in, A, s);
}

hipError_t launch_chirp_rows(const PassDesc& p, float2* A, hipStream_t s) {
  if (p.bH < 1 || p.bN % p.bH != 0) return hipErrorInvalidValue;
  switch (p.bN / p.bH) {
    case 256: return launch_rows<256>(p, A, s);
    case 512: return launch_rows<512>(p, A, s);
    case 1024: return launch_rows<1024>(p, A, s);
    case 2048: return launch_rows<2048>(p, A, s);
    case 4096: return launch_rows<4096>(p, A, s);
    case 8192: return launch_rows<8192>(p, A, s);
    case 16384: return launch_rows<16384>(p, A, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_chirp_out(const PassDesc& p, const float2* A, float2* out, hipStream_t s) {
  return p.wide ? launch_cols_h<false, true>(p, A, out, s)
                : launch_cols_h<false, false>(p, A, out, s);
}

}  // namespace lfft
