// Device body of the register-resident power-of-two FFT pass: one tile of
// W pencils of length L, P = 16 points per thread, Stockham stages of radix
// 2/4/8/16 in registers with padded LDS transposes between them, the natural
// gather fused into the first load and the natural scatter (plus the optional
// four-step twiddle and the 1/sqrt(m) scale) fused into the last store.
//
// Used by the one-launch-per-pass kernel and by the batched persistent kernel.
#pragma once
#include <hip/hip_runtime.h>

#include "fft_common.hpp"

namespace lfft {
namespace fastk {
using namespace dev;

__device__ __forceinline__ int phys(int e) { return e + (e >> 4); }

struct Pencil {
  long long b;
  int o, s;
  bool active;
};

// Butterfly geometry of pencil-local butterfly index bl in a stage.
struct BfGeom {
  int in0, in_step;    // positions of input i: in0 + i * in_step
  int out0, out_step;  // positions of output i: out0 + i * out_step
  int jm;              // j mod Ns (twiddle exponent)
};

__device__ __forceinline__ BfGeom geom(const StageDesc& st, int bl) {
  BfGeom g;
  const int lg_nr = st.lg_n - st.lg_r;
  const int l_lo = bl & (st.stride - 1);
  const int q = bl >> st.lg_stride;
  const int j = q & ((1 << lg_nr) - 1);
  const int l_hi = q >> lg_nr;
  const int base = (l_hi << (st.lg_n + st.lg_stride)) + l_lo;
  g.in0 = base + (j << st.lg_stride);
  g.in_step = 1 << (lg_nr + st.lg_stride);
  g.jm = j & (st.Ns - 1);
  const int idxD = ((j >> st.lg_Ns) << (st.lg_Ns + st.lg_r)) + g.jm;
  g.out0 = base + (idxD << st.lg_stride);
  g.out_step = 1 << (st.lg_Ns + st.lg_stride);
  return g;
}

// Last stage of a one-digit pencil, butterfly `bl` turned by `off`
// positions: with p = (bl + off) mod L the inputs of butterfly p mod Ns and
// the twiddles of exponent p (instead of p mod Ns) give the outputs
// p, p + Ns, ... mod L, the first one at p itself.
__device__ __forceinline__ BfGeom geom_turned(const StageDesc& st, int bl, int off) {
  BfGeom g;
  g.jm = (bl + off) & (st.n - 1);
  g.in0 = g.jm & (st.Ns - 1);
  g.in_step = st.Ns;          // n / radix = Ns in the last stage
  g.out0 = g.jm;
  g.out_step = st.Ns;
  return g;
}

// First stage of a one-digit pencil, butterfly `bl` turned by `off` positions
// on its inputs: with p = (bl + off) mod L value i is input (i + k) mod R of
// butterfly p mod (L / R), k = p / (L / R); load_first puts the inputs in order.
__device__ __forceinline__ int start_bf(const StageDesc& st, int bl, int off) {
  return off < 0 ? bl : (bl + off) & ((st.n >> st.lg_r) - 1);
}

// One side of a pencil: the signal's base pointer and 32-bit element
// offsets inside the signal (the planner keeps these lattices below 2^30
// points).
template <int MODE>
struct Addr {
  const float2* base;
  int lin;              // IDENTITY: o*L*S + s; LINEAR: To[o] + Ts[s]
  int cbase[4];         // NATURAL: To[o] (+) Ts[s]
};

template <int MODE>
__device__ __forceinline__ void addr_init(Addr<MODE>& A, const MapDesc& m, const float2* buf,
                                          const Pencil& pc, int L, int S) {
  A.base = buf + pc.b * m.bstride;
  if constexpr (MODE == MAP_IDENTITY) {
    A.lin = pc.o * L * S + pc.s;
  } else if constexpr (MODE == MAP_LINEAR) {
    A.lin = m.To[pc.o].x + m.Ts[pc.s].x;
  } else {
    A.cbase[0] = A.cbase[1] = A.cbase[2] = A.cbase[3] = 0;
    if (m.d == 2) {
      gadd2(m, A.cbase[0], A.cbase[1], m.To[pc.o]);
      gadd2(m, A.cbase[0], A.cbase[1], m.Ts[pc.s]);
    } else if (m.d == 3) {
      gadd3(m, A.cbase, m.To[pc.o]);
      gadd3(m, A.cbase, m.Ts[pc.s]);
    } else {
      gadd32(m, A.cbase, m.To[pc.o]);
      gadd32(m, A.cbase, m.Ts[pc.s]);
    }
  }
}

// Visit the element offsets of positions l0 + i*step, i < R.
template <int MODE, int R, class F>
__device__ __forceinline__ void for_positions(const Addr<MODE>& A, const MapDesc& m, int S, int l0,
                                              int step, F&& f) {
  if constexpr (MODE == MAP_IDENTITY) {
    const int a = A.lin + l0 * S;
#pragma unroll
    for (int i = 0; i < R; ++i) f(i, a + i * step * S);
  } else if constexpr (MODE == MAP_LINEAR) {
    // (an arithmetic progression, but with one constant in the place of the table
    // reads the stores come in denser bursts over the same memory channels:
    // [[4096, 1], [0, 4096]] into grid order 253 us, 238 so)
#pragma unroll
    for (int i = 0; i < R; ++i) f(i, A.lin + m.Tl[l0 + i * step].x);
  } else {
    const int4 D = m.Tl[step];
    if (m.d == 2) {
      int c0 = A.cbase[0], c1 = A.cbase[1];
      gadd2(m, c0, c1, m.Tl[l0]);
      const int h11 = m.H[1][1];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        f(i, c0 * h11 + c1);
        if (i + 1 < R) gadd2(m, c0, c1, D);
      }
    } else if (m.d == 3) {
      int c[4] = {A.cbase[0], A.cbase[1], A.cbase[2], 0};
      gadd3(m, c, m.Tl[l0]);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        f(i, nat_index3(m, c));
        if (i + 1 < R) gadd3(m, c, D);
      }
    } else {
      int c[4] = {A.cbase[0], A.cbase[1], A.cbase[2], A.cbase[3]};
      gadd32(m, c, m.Tl[l0]);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        f(i, nat_index_i(m, c));
        if (i + 1 < R) gadd32(m, c, D);
      }
    }
  }
}

template <int R>
__device__ __forceinline__ void dftR(float2* v, int sign) {
  dft_pow2<R>(v, sign);
}

template <int P, int R, int MIN, bool TURN>
__device__ __forceinline__ void load_first(float2* v, const PassDesc& p, const Addr<MIN>& A,
                                           int jt, int TPP, bool active, int off) {
  const StageDesc& st = p.st[0];
#pragma unroll
  for (int q = 0; q < P / R; ++q) {
    BfGeom g = geom(st, jt + TPP * q);
    if (off >= 0) g.in0 = (jt + TPP * q + off) & (st.n - 1);
    if (active) {
      for_positions<MIN, R>(A, p.in, p.S, g.in0, g.in_step,
                            [&](int i, int off) { v[q * R + i] = A.base[(unsigned)off]; });
    } else {
#pragma unroll
      for (int i = 0; i < R; ++i) v[q * R + i] = make_float2(0.f, 0.f);
    }
  }
  if constexpr (TURN)
    if (off >= 0) {
#pragma unroll
      for (int q = 0; q < P / R; ++q)
        rotate_by<R>(&v[q * R], ((jt + TPP * q + off) & (st.n - 1)) >> (st.lg_n - st.lg_r));
    }
}

// Base twiddles of a stage: for every butterfly of the thread, w^(2^k) for
// 2^k < R with w = exp(-2 pi i jm / (Ns R)), read from the FP64-built table
// of the digit.  Issued one stage ahead so their latency hides behind the
// LDS exchange.
// off >= 0: the turned last stage.
template <int P, int R>
__device__ __forceinline__ void prefetch_tw(float2* twb, const StageDesc& st, int jt, int TPP,
                                            int off) {
  constexpr int LG = R == 16 ? 4 : R == 8 ? 3 : R == 4 ? 2 : 1;
#pragma unroll
  for (int q = 0; q < P / R; ++q) {
    const int jm = off < 0 ? geom(st, jt + TPP * q).jm : geom_turned(st, jt + TPP * q, off).jm;
    const int tstep = jm << (st.lg_n - st.lg_Ns - st.lg_r);
#pragma unroll
    for (int k = 0; k < LG; ++k) twb[q * LG + k] = st.tw[(tstep << k) & (st.n - 1)];
  }
}

// Multiply input i of one butterfly by w^i, i = 1..R-1, building every power
// from the base powers w, w^2, w^4, w^8 with at most three products.
template <int R>
__device__ __forceinline__ void apply_tw(float2* x, const float2* b, int sign) {
  float2 pw[R];
  float2 b0 = b[0];
  if (sign > 0) b0.y = -b0.y;
  pw[1] = b0;
  if constexpr (R >= 4) {
    float2 b1 = b[1];
    if (sign > 0) b1.y = -b1.y;
    pw[2] = b1;
    pw[3] = c_mul(b0, b1);
  }
  if constexpr (R >= 8) {
    float2 b2 = b[2];
    if (sign > 0) b2.y = -b2.y;
    pw[4] = b2;
#pragma unroll
    for (int i = 5; i < 8; ++i) pw[i] = c_mul(pw[i - 4], b2);
  }
  if constexpr (R >= 16) {
    float2 b3 = b[3];
    if (sign > 0) b3.y = -b3.y;
    pw[8] = b3;
#pragma unroll
    for (int i = 9; i < 16; ++i) pw[i] = c_mul(pw[i - 8], b3);
  }
#pragma unroll
  for (int i = 1; i < R; ++i) x[i] = c_mul(x[i], pw[i]);
}

// tw: the stage has twiddles (Ns > 1; the first stage of a digit has none)
template <int P, int R>
__device__ __forceinline__ void compute_stage(float2* v, const float2* twb, int sign, bool tw) {
  constexpr int LG = R == 16 ? 4 : R == 8 ? 3 : R == 4 ? 2 : 1;
#pragma unroll
  for (int q = 0; q < P / R; ++q) {
    if (tw) apply_tw<R>(&v[q * R], &twb[q * LG], sign);
    dftR<R>(&v[q * R], sign);
  }
}

// LDS element of pencil-local position l of tile pencil w: padded by one
// element in 16; PR is the padded length of a row.
template <bool COLS>
__device__ __forceinline__ int lds_e(int l, int w, int W, int PR) {
  return COLS ? phys(l * W + w) : w * PR + phys(l);
}

// Visit the LDS elements of positions l0 + i step, i < R.  The padding keeps
// them an arithmetic progression when a step moves by whole 16-element groups
// or when the R positions lie within one (a first stage's outputs, R of them
// from a multiple of R): one addition per element then.
template <int R, bool COLS, class F>
__device__ __forceinline__ void for_lds(int l0, int step, int w, int W, int PR, F&& f) {
  const int d = COLS ? step * W : step;
  if ((d & 15) == 0 || (!COLS && step == 1)) {
    const int e0 = lds_e<COLS>(l0, w, W, PR), de = d + (d >> 4);
#pragma unroll
    for (int i = 0; i < R; ++i) f(i, e0 + i * de);
  } else {
#pragma unroll
    for (int i = 0; i < R; ++i) f(i, lds_e<COLS>(l0 + i * step, w, W, PR));
  }
}

template <int P, int R, bool COLS, int PART>
__device__ __forceinline__ void lds_write(const float2* v, void* lds, const StageDesc& st, int jt,
                                          int TPP, int w, int W, int PR, int off) {
#pragma unroll
  for (int q = 0; q < P / R; ++q) {
    const BfGeom g = geom(st, start_bf(st, jt + TPP * q, off));
    for_lds<R, COLS>(g.out0, g.out_step, w, W, PR, [&](int i, int e) {
      if constexpr (PART == 0)
        static_cast<float2*>(lds)[e] = v[q * R + i];
      else if constexpr (PART == 1)
        static_cast<float*>(lds)[e] = v[q * R + i].x;
      else
        static_cast<float*>(lds)[e] = v[q * R + i].y;
    });
  }
}

template <int P, int R, bool COLS, int PART>
__device__ __forceinline__ void lds_read(float2* v, const void* lds, const StageDesc& st, int jt,
                                         int TPP, int w, int W, int PR, int off) {
#pragma unroll
  for (int q = 0; q < P / R; ++q) {
    const BfGeom g = off < 0 ? geom(st, jt + TPP * q) : geom_turned(st, jt + TPP * q, off);
    for_lds<R, COLS>(g.in0, g.in_step, w, W, PR, [&](int i, int e) {
      if constexpr (PART == 0)
        v[q * R + i] = static_cast<const float2*>(lds)[e];
      else if constexpr (PART == 1)
        v[q * R + i].x = static_cast<const float*>(lds)[e];
      else
        v[q * R + i].y = static_cast<const float*>(lds)[e];
    });
  }
}

#define LFFT_RADIX_SWITCH(R_, ...)                         \
  switch (R_) {                                            \
    case 2: { constexpr int RR = 2; __VA_ARGS__; } break;   \
    case 4: { constexpr int RR = 4; __VA_ARGS__; } break;   \
    case 8: { constexpr int RR = 8; __VA_ARGS__; } break;   \
    default: { constexpr int RR = 16; __VA_ARGS__; } break; \
  }

template <int P, int R, int MOUT>
__device__ __forceinline__ void store_last_r(const float2* v, const PassDesc& p,
                                             const Addr<MOUT>& A, int jt, int TPP,
                                             const Pencil& pc, int off0) {
  const StageDesc& st = p.st[p.nst - 1];
  float2* out = const_cast<float2*>(A.base);
  // (read once: for all the compiler knows, the stores below change them)
  const float scale = p.scale, scale_lo = p.scale_lo;
  const bool scaled = scale != 1.0f, post = p.post != 0;
  // four-step twiddle exponent (l mod post_lmod) * lo, lo fixed per pencil
  const unsigned lo = post ? post_lo(p, pc.s) : 0u;
#pragma unroll
  for (int q = 0; q < P / R; ++q) {
    const BfGeom g = off0 < 0 ? geom(st, jt + TPP * q) : geom_turned(st, jt + TPP * q, off0);
    for_positions<MOUT, R>(A, p.out, p.S, g.out0, g.out_step, [&](int i, int off) {
      float2 x = v[q * R + i];
      if (post) {
        const unsigned l = (unsigned)(g.out0 + i * g.out_step) & (unsigned)(p.post_lmod - 1);
        x = c_mul(x, post_twiddle(p, l * lo));
      }
      if (scaled) x = c_scale(x, scale, scale_lo);
      out[(unsigned)off] = x;
    });
  }
}

template <int P, int MOUT>
__device__ __forceinline__ void store_last(const float2* v, const PassDesc& p, const Addr<MOUT>& A,
                                           int jt, int TPP, const Pencil& pc, int off) {
  LFFT_RADIX_SWITCH(p.st[p.nst - 1].radix, (store_last_r<P, RR, MOUT>(v, p, A, jt, TPP, pc, off)));
}

// Pencil `pen` of the pass (inactive beyond the last one), rows in the order
// of `chain` if there is one; off: its position offset there.
__device__ __forceinline__ Pencil pencil_at(const PassDesc& p, long long pen, const int2* chain,
                                            int& off) {
  Pencil pc;
  pc.active = pen < p.batch * (long long)p.O * p.S;
  const long long pp = pc.active ? pen : 0;
  const long long bo = pp / p.S;
  pc.s = (int)(pp - bo * p.S);
  pc.b = bo / p.O;
  pc.o = (int)(bo - pc.b * p.O);
  if (chain) {
    const int2 c = chain[pc.o];
    pc.o = c.x;
    off = c.y;
  }
  return pc;
}

// Process tile `tile` of pass p with NT = W * L / P threads (tid < NT);
// lds holds (W*L + W*L/16 + kTilePad) float2 (SPLIT: floats).
//
// Row tiles of a last pass: natural neighbours lie in different rows unless
// the axis is aligned with the natural order, and a thread order along the
// row writes single elements to lines of their own.  The planner therefore
// gathers the rows of W natural neighbours in one tile (chain: reading whole
// rows costs the same in any order), and the last stage runs with
// neighbouring threads on neighbouring rows, each row turned by the position
// of its neighbour, so that a wave writes runs of W elements.  The change of
// thread order rides on the last LDS exchange and the turn on the twiddles,
// so neither costs anything.  Column tiles only reorder their own columns; on
// the input side of a first pass the turn costs log2(R) selects per value and,
// unlike a product with the root that the turn leaves on the outputs, no
// rounding (mask gradients of 16 x 2^20 points were up to 8% further from 64
// bits with it).  The rows' LDS pitch is 32 / W elements modulo 32 then, which
// spreads those reads over all banks.
constexpr int kTilePad = 33;

// TURN: the input side may have a chain (column tiles).
template <int P, bool COLS, bool SPLIT, int MIN, int MOUT, bool TURN>
__device__ __forceinline__ void fast_tile(const PassDesc& p, long long tile, int tid,
                                          const float2* __restrict__ in,
                                          float2* __restrict__ out, void* lds) {
  const int L = p.L, S = p.S, W = p.W;
  const int TPP = L / P;
  int w, jt;
  if (COLS) {
    w = tid % W;
    jt = tid / W;
  } else {
    w = tid / TPP;
    jt = tid - w * TPP;
  }
  const bool turn = !COLS && !SPLIT && MOUT != MAP_IDENTITY && W > 1 && p.out.across;
  const int PR = phys(L) + (turn && L >= 512 ? 32 / W : 0);
  const int2* chain = !COLS && MOUT == MAP_NATURAL ? p.out.chain : nullptr;
  int off = -1, unused = -1;   // position offset of the last stage (-1: none)
  static_assert(!TURN || (COLS && MIN == MAP_NATURAL && MOUT != MAP_NATURAL), "first pass");
  int off_cols = -1, off_in = -1;
  if (COLS && MOUT == MAP_NATURAL) {
    if (p.out.chain) {
      const int2 c = p.out.chain[w];
      w = c.x;
      off_cols = c.y;
    }
  } else if (TURN && p.in.chain) {
    const int2 c = p.in.chain[w];
    w = c.x;
    off_in = c.y;
  }
  Pencil pc = pencil_at(p, tile * W + w, chain, unused);
  float2 v[P];
  {
    Addr<MIN> A;
    addr_init<MIN>(A, p.in, in, pc, L, S);
    LFFT_RADIX_SWITCH(p.st[0].radix, (load_first<P, RR, MIN, TURN>(v, p, A, jt, TPP, pc.active, off_in)));
  }
  float2 twb[8];
  if (p.st[0].Ns > 1)
    LFFT_RADIX_SWITCH(p.st[0].radix, (prefetch_tw<P, RR>(twb, p.st[0], jt, TPP, -1)));
  for (int si = 0; si < p.nst; ++si) {
    const StageDesc& st = p.st[si];
    LFFT_RADIX_SWITCH(st.radix, (compute_stage<P, RR>(v, twb, p.sign, st.Ns > 1)));
    if (si + 1 < p.nst) {
      const StageDesc& nx = p.st[si + 1];
      const int w0 = w, j0 = jt;
      if (COLS && si + 2 == p.nst) off = off_cols;
      if (turn && si + 2 == p.nst) {
        w = tid % W;
        jt = tid / W;
        pc = pencil_at(p, tile * W + w, chain, off);
      }
      if (nx.Ns > 1) LFFT_RADIX_SWITCH(nx.radix, (prefetch_tw<P, RR>(twb, nx, jt, TPP, off)));
      if constexpr (!SPLIT) {
        LFFT_RADIX_SWITCH(st.radix, (lds_write<P, RR, COLS, 0>(v, lds, st, j0, TPP, w0, W, PR, si ? -1 : off_in)));
        __syncthreads();
        LFFT_RADIX_SWITCH(nx.radix, (lds_read<P, RR, COLS, 0>(v, lds, nx, jt, TPP, w, W, PR, off)));
        __syncthreads();
      } else {
        LFFT_RADIX_SWITCH(st.radix, (lds_write<P, RR, COLS, 1>(v, lds, st, j0, TPP, w0, W, PR, si ? -1 : off_in)));
        __syncthreads();
        LFFT_RADIX_SWITCH(nx.radix, (lds_read<P, RR, COLS, 1>(v, lds, nx, jt, TPP, w, W, PR, off)));
        __syncthreads();
        LFFT_RADIX_SWITCH(st.radix, (lds_write<P, RR, COLS, 2>(v, lds, st, j0, TPP, w0, W, PR, si ? -1 : off_in)));
        __syncthreads();
        LFFT_RADIX_SWITCH(nx.radix, (lds_read<P, RR, COLS, 2>(v, lds, nx, jt, TPP, w, W, PR, off)));
        __syncthreads();
      }
    }
  }
  if (pc.active) {
    Addr<MOUT> A;
    addr_init<MOUT>(A, p.out, out, pc, L, S);
    store_last<P, MOUT>(v, p, A, jt, TPP, pc, off);
  }
}

}  // namespace fastk
}  // namespace lfft
