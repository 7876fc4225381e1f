// Mixed-radix FFT pass for gfx950: any pencil length up to 8192.  One
// workgroup owns a tile of TP pencils that moves between two LDS buffers, one
// Stockham stage per move; radices 2 .. 16 and the primes 17 .. 31 run in
// registers, larger primes as sums shared by all threads: a few of the longest
// digits, and inside pencils of several digits (the others are chirp-z passes).
//
// The first stage reads its butterflies straight from the input order and the
// last one writes straight to the output order, through the planner's maps
// (Section 3 bases, Theorem 1 of Section 4.1): the R positions of a butterfly
// are an arithmetic progression in one digit, so their natural coordinates
// follow by repeated group addition of one constant, and neither order is
// ever materialised.  Neighbouring threads take neighbouring pencils or
// neighbouring positions, chosen per side by the planner for the shorter
// memory step.
//
// Bound by latency and by the vector ALUs, not by HBM: a stage is one LDS
// round trip and a barrier, so stages are few and wide, and tiles are small:
// at most 4096 elements, 70 KB for both buffers and two workgroups of eight
// waves per CU (columns of 2 or 3 points 104 KB with their padding, single
// pencils near 8192 points 139 KB, one workgroup per CU).  All index splits are multiplications by precomputed
// reciprocals: with the integer divisions (64-bit for every twiddle) of a
// direct formulation, and single threads summing a prime's inputs, 1088
// points (8 x 17) took 111 us and 8 x 135135 points 494 us; now 9 and 32 us
// (13 and 35 before the descriptor's lines were fetched together).
#include <hip/hip_runtime.h>

#include <atomic>

#include "dft_small.hpp"
#include "kernels.hpp"
#include "pass_addr.hpp"

namespace lfft {
namespace {
using namespace dev;

constexpr int kPassThreads = 1024;

// The descriptor through the kernel argument segment (scalar loads).  Each
// stage takes a fresh view of it: the compiler would otherwise hoist every
// field that any radix reads to the kernel's entry and spill them.
typedef const __attribute__((address_space(4))) PassDesc* PassArg;
__device__ __forceinline__ const PassDesc& fresh(PassArg k) {
  asm volatile("" : "+s"(k));
  return *(const PassDesc*)k;
}

__device__ __forceinline__ int mphys(int e) { return e + (e >> 4); }

// Butterfly index -> tile pencil and pencil-local butterfly, with
// neighbouring indices across the pencils or along one.
__device__ __forceinline__ void split_bf(const PassDesc& p, FastDiv per, int nper, bool across,
                                         unsigned bf, int& w, unsigned& q) {
  if (across) {
    const unsigned t = fast_div(bf, p.f_TP);
    w = (int)(bf - t * (unsigned)p.TP);
    q = t;
  } else {
    w = (int)fast_div(bf, per);
    q = bf - (unsigned)w * (unsigned)nper;
  }
}

// multiply input i by w^i (primes above 16: every power from the table)
template <int R>
__device__ __forceinline__ void apply_powers(float2* v, const float2* tw, unsigned e, int sign) {
  if constexpr (R > 16) {
#pragma unroll
    for (int i = 1; i < R; ++i) v[i] = c_mul(v[i], tw_lookup(tw, (long long)(e * (unsigned)i), sign));
  } else {
    float2 b[tw_bases(R)];
#pragma unroll
    for (int k = 0; k < tw_bases(R); ++k)
      b[k] = tw_lookup(tw, (long long)(e * (unsigned)tw_exponent(k)), sign);
    apply_twiddles<R>(v, b);
  }
}

// One Stockham stage of radix R over the tile.  GIN / GOUT: the inputs come
// from the input order, the outputs go to the output order.
template <int R, bool GIN, bool GOUT>
__device__ __forceinline__ void stage(PassArg arg, int si, const TileOf& t,
                                      const float2* __restrict__ in, float2* __restrict__ out,
                                      const float2* A, float2* B) {
  const PassDesc& p = fresh(arg);
  const StageDesc& st = p.st[si];
  const int n = st.n, stride = st.stride, Ns = st.Ns;
  const int nr = n / R, per = p.L / R;
  const bool across = GIN ? p.in.across : GOUT ? p.out.across : p.ls != 1;
  const unsigned total = (unsigned)(across ? p.TP * per : t.n * per);
  const bool whole = stride == 1 && n == p.L;   // one digit: no outer or inner index
  for (unsigned bf = threadIdx.x; bf < total; bf += blockDim.x) {
    int w;
    unsigned q;
    split_bf(p, st.f_per, per, across, bf, w, q);
    if (w >= t.n) continue;
    unsigned l_lo = 0, j = q, l_hi = 0;
    if (!whole) {
      const unsigned a = fast_div(q, st.f_stride);
      l_lo = q - a * (unsigned)stride;
      l_hi = fast_div(a, st.f_nr);
      j = a - l_hi * (unsigned)nr;
    }
    const unsigned jd = fast_div(j, st.f_Ns);
    const unsigned jm = j - jd * (unsigned)Ns;
    const int base = (int)(l_hi * (unsigned)(n * stride) + l_lo);
    const int in0 = base + (int)j * stride, in_step = nr * stride;
    const int out0 = base + (int)(jd * (unsigned)(Ns * R) + jm) * stride, out_step = Ns * stride;
    Pencil pc{0, 0, 0};
    if (GIN || GOUT) pc = pencil_of(p, t, w);
    float2 v[R];
    if constexpr (GIN) {
      unsigned off[R];
      offsets<R, false>(p, p.in, pc, in0, in_step, off);
      const float2* src = in + pc.b * p.in.bstride;
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = src[off[i]];
    } else {
      const int e0 = in0 * p.ls + w * p.ws, es = in_step * p.ls;
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = A[mphys(e0 + i * es)];
    }
    if (Ns > 1) apply_powers<R>(v, dev_ptr(st.tw), (unsigned)(n / (Ns * R)) * jm, p.sign);
    if constexpr (GOUT) {
      dft_small<R>(v, p.sign);
      unsigned off[R];
      offsets<R, false>(p, p.out, pc, out0, out_step, off);
      float2* dst = out + pc.b * p.out.bstride;
      if (p.post) {
        // the stage's digit is the last one (stride 1) or l's position in it
        // does not change over the butterfly
        const unsigned lo = post_lo(p, pc.s);
        const unsigned x0 = post_pos(p, (unsigned)out0) * lo;
        const unsigned xs = stride == 1 ? (unsigned)Ns * lo : 0u;
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = c_mul(v[i], post_twiddle(p, x0 + (unsigned)i * xs));
      }
      const float scale = p.scale, scale_lo = p.scale_lo;
#pragma unroll
      for (int i = 0; i < R; ++i) dst[off[i]] = c_scale(v[i], scale, scale_lo);
    } else {
      const int e0 = out0 * p.ls + w * p.ws, es = out_step * p.ls;
      if constexpr (R > 16) {
        dft_odd_emit<R>(v, p.sign, [&](int k, float2 x) { B[mphys(e0 + k * es)] = x; });
      } else {
        dft_small<R>(v, p.sign);
#pragma unroll
        for (int i = 0; i < R; ++i) B[mphys(e0 + i * es)] = v[i];
      }
    }
  }
}

// A stage of a prime radix R, 37 .. kMaxDirect: the inputs with their
// twiddles are folded in place into x_j + x_{R-j} (at j) and x_j - x_{R-j} (at
// R - j), then one thread forms the outputs k and R - k from sums of (R - 1) / 2
// products each, over the R roots in LDS.  Bound by the vector ALUs of the few
// CUs that such a pass fills: 13 signals of 2368 = 64 x 37 points take 19.8 us.
__device__ __forceinline__ void stage_prime(PassArg arg, int si, const TileOf& t, float2* A,
                                            float2* B, float2* roots) {
  const PassDesc& p = fresh(arg);
  const StageDesc& st = p.st[si];
  const int R = st.radix, n = st.n, stride = st.stride, Ns = st.Ns;
  const int nr = n / R, h = (R - 1) / 2, per = p.L / R;
  const float2* tw = dev_ptr(st.tw);
  for (int k = threadIdx.x; k < R; k += blockDim.x) roots[k] = tw[k * nr];
  // butterfly bf: first input, twiddle exponent, first output; steps in0s, out0s
  auto place = [&](unsigned bf, int& in0, int& e, int& out0) {
    const int w = (int)fast_div(bf, st.f_per);
    const unsigned q = bf - (unsigned)w * (unsigned)per;
    const unsigned a = fast_div(q, st.f_stride), l_lo = q - a * (unsigned)stride;
    const unsigned l_hi = fast_div(a, st.f_nr), j = a - l_hi * (unsigned)nr;
    const unsigned jd = fast_div(j, st.f_Ns), jm = j - jd * (unsigned)Ns;
    const int base = (int)(l_hi * (unsigned)(n * stride) + l_lo);
    in0 = (base + (int)j * stride) * p.ls + w * p.ws;
    e = n / (Ns * R) * (int)jm;
    out0 = (base + (int)(jd * (unsigned)(Ns * R) + jm) * stride) * p.ls + w * p.ws;
  };
  const int in_step = nr * stride * p.ls, out_step = Ns * stride * p.ls;
  const unsigned bfs = (unsigned)(t.n * per);
  for (unsigned x = threadIdx.x; x < bfs * (unsigned)h; x += blockDim.x) {
    const unsigned bf = x / (unsigned)h;
    const int j = (int)(x - bf * (unsigned)h) + 1;
    int in0, e, out0;
    place(bf, in0, e, out0);
    const int pa = mphys(in0 + j * in_step), pb = mphys(in0 + (R - j) * in_step);
    float2 a = A[pa], b = A[pb];
    if (Ns > 1) {
      a = c_mul(a, tw_lookup(tw, e * j, p.sign));
      b = c_mul(b, tw_lookup(tw, e * (R - j), p.sign));
    }
    A[pa] = c_add(a, b);
    A[pb] = c_sub(a, b);
  }
  __syncthreads();
  for (unsigned x = threadIdx.x; x < bfs * (unsigned)(h + 1); x += blockDim.x) {
    const unsigned bf = x / (unsigned)(h + 1);
    const int k = (int)(x - bf * (unsigned)(h + 1));
    int in0, e, out0;
    place(bf, in0, e, out0);
    float2 a = A[mphys(in0)], b = make_float2(0.f, 0.f);
    int r = 0;
#pragma unroll 4
    for (int j = 1; j <= h; ++j) {
      r += k;
      r -= r >= R ? R : 0;
      const float2 w = roots[r];      // cos, -sin
      const float2 s = A[mphys(in0 + j * in_step)], d = A[mphys(in0 + (R - j) * in_step)];
      a.x += w.x * s.x;
      a.y += w.x * s.y;
      b.x -= w.y * d.x;
      b.y -= w.y * d.y;
    }
    b = c_muli(b, p.sign);
    B[mphys(out0 + k * out_step)] = c_add(a, b);
    if (k) B[mphys(out0 + (R - k) * out_step)] = c_sub(a, b);
  }
}

// A stage of any radix: one thread per output, the inputs from LDS (lanes of
// one butterfly read the same word), the root's exponent kept by addition.
__device__ __forceinline__ void stage_sum(PassArg arg, int si, const TileOf& t,
                                       const float2* A, float2* B) {
  const PassDesc& p = fresh(arg);
  const StageDesc& st = p.st[si];
  const int R = st.radix, n = st.n, stride = st.stride, Ns = st.Ns;
  const int nr = n / R;
  const unsigned total = (unsigned)t.n * (unsigned)p.L;
  for (unsigned e = threadIdx.x; e < total; e += blockDim.x) {
    const int w = (int)fast_div(e, p.f_L);
    const int l = (int)(e - (unsigned)w * (unsigned)p.L);
    // output position l: digits (l_hi, idx, l_lo) with
    // idx = jd Ns R + k Ns + jm
    const int a = l / stride, l_lo = l - a * stride;
    const int l_hi = a / n, idx = a - l_hi * n;
    const int jd = idx / (Ns * R), rem = idx - jd * (Ns * R);
    const int k = rem / Ns, jm = rem - k * Ns;
    const int j = jd * Ns + jm;
    const int base = l_hi * n * stride + l_lo;
    // input i carries exp(sign 2 pi i (tstep i + nr ((i k) mod R)) / n)
    const int inc = (int)(((long long)(n / (Ns * R)) * jm + (long long)nr * k) % n);
    int x = 0;
    float2 acc = make_float2(0.f, 0.f);
    int pos = (base + j * stride) * p.ls + w * p.ws;
    const int step = nr * stride * p.ls;
    for (int i = 0; i < R; ++i) {
      acc = c_add(acc, c_mul(A[mphys(pos)], tw_lookup(dev_ptr(st.tw), x, p.sign)));
      pos += step;
      x += inc;
      x -= x >= n ? n : 0;
    }
    B[mphys(l * p.ls + w * p.ws)] = acc;
  }
}

#define LFFT_SMALL_RADIX(X) \
  X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#define LFFT_MIXED_PRIME(X) X(17) X(19) X(23) X(29) X(31)

// WIDE: 2^30 points and more, 64-bit coordinates; the input and the output
// then move through LDS one element at a time (registers).
template <bool WIDE>
__global__ void __launch_bounds__(kPassThreads)
    fft_mixed_kernel(PassDesc, const float2* __restrict__ in, float2* __restrict__ out) {
  extern __shared__ float2 lds[];
  touch_args<sizeof(PassDesc)>();
  const PassArg arg = (PassArg)__builtin_amdgcn_kernarg_segment_ptr();
  const PassDesc& p = *(const PassDesc*)arg;
  const int half = mphys(p.ls == 1 ? p.TP * p.ws : p.L * p.ls) + 1;
  float2* A = lds;
  float2* B = lds + half;
  const TileOf t = tile_of_pencils(p, xcd_tile(blockIdx.x, gridDim.x) * p.TP, p.TP);

  const int last = p.nst - 1;
  const bool gin = !WIDE && p.nst > 0 && p.st[0].radix <= 16;
  const bool gout = !WIDE && p.nst > 0 && p.st[last].radix <= 16;
  if (!gin) {
    const bool across = p.in.across;
    const unsigned total = (unsigned)((across ? p.TP : t.n) * p.L);
    for (unsigned e = threadIdx.x; e < total; e += blockDim.x) {
      int w;
      unsigned l;
      split_bf(p, p.f_L, p.L, across, e, w, l);
      if (w >= t.n) continue;
      const Pencil pc = pencil_of(p, t, w);
      unsigned off[1];
      offsets<1, WIDE>(p, p.in, pc, (int)l, 0, off);
      A[mphys((int)l * p.ls + w * p.ws)] = in[pc.b * p.in.bstride + off[0]];
    }
    __syncthreads();
  }
  for (int si = 0; si < p.nst; ++si) {
    const int radix = p.st[si].radix;
    const bool first = si == 0 && gin, end = si == last && gout;
    bool done = false;
    if constexpr (!WIDE) {
      if (first && end) {
        switch (radix) {
#define X(R) case R: stage<R, true, true>(arg, si, t, in, out, A, B); break;
          LFFT_SMALL_RADIX(X)
#undef X
        }
        return;
      }
      if (first) {
        done = true;
        switch (radix) {
#define X(R) case R: stage<R, true, false>(arg, si, t, in, out, A, B); break;
          LFFT_SMALL_RADIX(X)
#undef X
        }
      } else if (end) {
        switch (radix) {
#define X(R) case R: stage<R, false, true>(arg, si, t, in, out, A, B); break;
          LFFT_SMALL_RADIX(X)
#undef X
        }
        return;
      }
    }
    if (!done) {
      switch (radix) {
#define X(R) case R: stage<R, false, false>(arg, si, t, in, out, A, B); break;
        LFFT_SMALL_RADIX(X)
        LFFT_MIXED_PRIME(X)
#undef X
        default:
          if (radix <= kMaxDirect)
            stage_prime(arg, si, t, A, B, lds + 2 * half);
          else
            stage_sum(arg, si, t, A, B);
          break;
      }
    }
    __syncthreads();
    float2* x = A;
    A = B;
    B = x;
  }
  const bool across = p.out.across;
  const unsigned total = (unsigned)((across ? p.TP : t.n) * p.L);
  for (unsigned e = threadIdx.x; e < total; e += blockDim.x) {
    int w;
    unsigned l;
    split_bf(p, p.f_L, p.L, across, e, w, l);
    if (w >= t.n) continue;
    const Pencil pc = pencil_of(p, t, w);
    unsigned off[1];
    offsets<1, WIDE>(p, p.out, pc, (int)l, 0, off);
    float2 v = A[mphys((int)l * p.ls + w * p.ws)];
    if (p.post) v = c_mul(v, post_twiddle(p, post_pos(p, l) * post_lo(p, pc.s)));
    out[pc.b * p.out.bstride + off[0]] = c_scale(v, p.scale, p.scale_lo);
  }
}

template <bool WIDE>
hipError_t launch_mixed_t(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  static std::atomic<bool> attr{false};
  if (!attr.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)fft_mixed_kernel<WIDE>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr.store(true, std::memory_order_release);
  }
  const long long npen = p.batch * (long long)p.O * p.S;
  const long long tiles = (npen + p.TP - 1) / p.TP;
  const int span = p.ls == 1 ? p.TP * p.ws : p.L * p.ls;
  bool prime = false;
  for (int i = 0; i < p.nst; ++i) prime = prime || p.st[i].radix > 31;
  const size_t lds = (size_t)(2 * (span + span / 16 + 1) + (prime ? kMaxDirect : 0)) * sizeof(float2);
  if (tiles <= 0) return hipSuccess;
  if (tiles > 0x7fffffffLL || lds > 160 * 1024 || p.NT < 64 || p.NT > kPassThreads)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(fft_mixed_kernel<WIDE>, dim3((unsigned)tiles), dim3(p.NT), lds, s, p, in, out);
  return hipGetLastError();
}

}  // namespace

const char* pass_kernel_name(const PassDesc& p) {
  if (p.kind >= 4) return chirp_kernel_name(p);
  if (p.kind == 3) return mfma_kernel_name(p);
  if (p.kind == 2) return stream_kernel_name(p);
  return p.kind == 1 ? fast_kernel_name(p)
                     : p.wide ? "fft_mixed_kernel<true>" : "fft_mixed_kernel<false>";
}

hipError_t launch_pass(const PassDesc& p, const float2* in, float2* out, hipStream_t s) {
  if (p.kind == 5) return launch_chirp_tile(p, in, out, s);
  if (p.kind == 3) return launch_mfma_pass(p, in, out, s);
  if (p.kind == 2) return launch_stream_pass(p, in, out, s);
  if (p.kind == 1) return launch_fast_pass(p, in, out, s);
  return p.wide ? launch_mixed_t<true>(p, in, out, s) : launch_mixed_t<false>(p, in, out, s);
}

}  // namespace lfft
