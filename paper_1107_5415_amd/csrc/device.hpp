// Plain-old-data descriptors handed from the host planner to the gfx950
// kernels by value.  All pointers are device pointers into the plan's table
// blob.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace lfft {

// Stages of one pass: within a digit of length n any two radices multiply to
// more than 16, so a pencil of at most 8192 points in up to seven digits
// needs no more.
constexpr int kMaxStages = 12;

// floor(n / d) for 0 <= n < 2^31 as (n * mag) >> (31 + sh), with
// sh = ceil(log2 d) and mag = floor(2^(31 + sh) / d) + 1 < 2^32 (division by
// an invariant integer through multiplication; the rounding error of the
// scaled reciprocal stays below 1/d for n < 2^31).
struct FastDiv {
  unsigned mag;
  int sh;
};

__host__ __device__ __forceinline__ unsigned fast_div(unsigned n, FastDiv f) {
  return (unsigned)(((unsigned long long)n * f.mag) >> (31 + f.sh));
}

// How a pass addresses the buffer on one side.
//   IDENTITY : the internal grid layout, index = ((b*O + o)*L + l)*S + s
//   LINEAR   : separable offsets, index = b*bstride + To[o].x + Tl[l].x + Ts[s].x
//   NATURAL  : natural residue box of a lattice (column Hermite form H):
//              coords = To[o] (+) Tl[l] (+) Ts[s]  (group sum in Z^d / H Z^d),
//              index  = b*bstride + sum_i coords_i * box_stride_i
enum MapMode : int { MAP_IDENTITY = 0, MAP_LINEAR = 1, MAP_NATURAL = 2 };

struct MapDesc {
  int mode;
  int d;
  int across;                 // neighbouring threads on neighbouring pencils (0: on
                              // neighbouring positions of one pencil); not in the
                              // streaming and split-BF16 kernels
  int H[4][4];
  long long box_stride[4];
  long long bstride;          // batch stride in elements (LINEAR / NATURAL)
  const int4* To;
  const int4* Tl;
  const int4* Ts;
  // register-resident kernel, last pass over rows: chain[t W + w] = (row,
  // position) of tile t's w-th row and of the w-th of W consecutive natural
  // elements, the first of which lies at position 0 of the tile's first row (or
  // of several shorter runs);
  // streaming and register-resident kernels, last pass over columns:
  // chain[w] = (column, position) likewise inside every tile of W columns, in
  // runs, and on the input side of a first pass over columns (NULL: in order)
  const int2* chain;
  // LINEAR, streaming kernel, last pass over columns: the columns are groups x
  // low indices of a four-step axis whose values lie side by side over the
  // groups (0: no such axis)
  int groups;
};

// One Stockham stage: radix r on the pass digit of length n whose stride
// inside the pencil index l is `stride`; Ns is the product of the radices
// already applied to that digit.  tw[k] = exp(-2 pi i k / n), k in [0, n).
struct StageDesc {
  int radix;
  int n;
  int stride;
  int Ns;
  const float2* tw;
  // base-2 logarithms (power-of-two stages only, used by the fast kernel)
  int lg_r, lg_n, lg_stride, lg_Ns;
  // mixed-radix kernel: divisions by the stride, by n / radix, by Ns and by
  // the butterflies of one pencil, L / radix
  FastDiv f_stride, f_nr, f_Ns, f_per;
};

struct PassDesc {
  int kind;                   // 0 mixed-radix, 1 register-resident power-of-two, 2 streaming,
                              // 3 split-BF16 MFMA, 4 chirp-z (a long axis),
                              // 5 chirp-z on chip (one digit of at most 8192 points)
  int P;                      // fast kernel: points per thread (16)
  int W;                      // fast kernel: pencils per workgroup
  int split;                  // fast kernel: exchange real and imaginary parts separately
  long long batch;            // number of signals
  int O, L, S;                // per-signal outer count, pencil length, inner count
  // mixed-radix kernel: pencils per tile, threads, the LDS position of pencil
  // position l of tile pencil w (l * ls + w * ws), 64-bit coordinates, and
  // its divisions
  int TP, NT;
  int ls, ws;
  int wide;
  FastDiv f_TP, f_S, f_OS, f_L, f_lmod;
  int nst;
  StageDesc st[kMaxStages];
  int sign;                   // -1 forward, +1 inverse
  float scale, scale_lo;      // applied when storing: their sum
  // streaming kernel, last pass of a natural-order transform whose rows
  // pencils write whole aligned rows of the caller's output: stores marked
  // non-temporal, so that they do not evict the input and the intermediate
  // grid from the caches; its loads of the intermediate grid (whole rows,
  // dead once read) are non-temporal too
  int stream_out;
  // streaming kernel, first pass reading whole aligned rows of the caller's
  // natural-order input (read once by the call): loads marked non-temporal,
  // so that the intermediate grid stays in the caches for the next pass
  int stream_in;
  // four-step twiddle after the stages: x = (l mod post_lmod) * lo with
  // lo = (s / lo_div) % lo_n, below postN = post_lmod lo_n, factor exp(sign 2 pi i x / postN)
  // from the two-level table tw_hi[x >> 12] * tw_lo[x & 4095]; the high digit
  // is the last (fastest) digit of the pencil, of length post_lmod
  int post;
  int postN;
  int post_lmod;
  int lo_div;
  int lo_n;
  FastDiv f_lodiv, f_lon;
  const float2* tw_hi;
  const float2* tw_lo;
  // chirp-z passes: the axis or digit of length L as a cyclic convolution of
  // length bN (a power of two >= 2L - 1); chirp[j] = exp(-pi i j^2 / L), bhat =
  // the DFT of the convolution kernel conj(chirp) over bN (both conjugated
  // for sign +1).  Kind 4 (three launches): bN = bH R, element n = a R + c,
  // bhat in the order (k mod bH, k / bH); tables exp(-2 pi i k / n) of the
  // columns (tw_col, n = bH) and the rows (tw_row, n = R), and two-level for
  // bN (cv_hi, cv_lo).  Kind 5 (one launch): tw_row for n = bN.
  int bN, bH;
  const float2* chirp;
  const float2* bhat;
  const float2* tw_row;
  const float2* tw_col;
  const float2* cv_hi;
  const float2* cv_lo;
  MapDesc in, out;
};

// One pass of one lattice in the batched persistent launch.  Buffers are
// selected by index (0 caller input, 1 caller output, 2 workspace) so the
// descriptors do not depend on the call's pointers.
struct BatchPass {
  PassDesc pd;                // batch 1, maps and batch strides resolved
  long long in_off, out_off;  // element offsets of the lattice's signal
  int in_buf, out_buf;
  int variant;                // body: BATCH_ROWS_NN .. BATCH_COLS_IN
};

enum BatchVariant : int {
  BATCH_ROWS_NN = 0,          // contiguous pencils, natural in, natural out (one-pass lattice)
  BATCH_ROWS_NI = 1,          // contiguous pencils, natural in, grid out
  BATCH_COLS_NI = 2,          // strided pencils, natural in, grid out
  BATCH_ROWS_IN = 3,          // contiguous pencils, grid in, natural out
  BATCH_COLS_IN = 4,          // strided pencils, grid in, natural out
};

// One level of the Fourier-domain wavelet split (natural orders).
struct SplitDesc {
  long long mM;               // |det M_l| (points of the level)
  long long mN;               // |det N_l| = mM / 2
  int d;
  int KN[4];                  // natural box of N_l^T (Hermite diagonal)
  long long kstride[4];
  int HM[4][4];               // column Hermite form of M_l^T
  long long hstride[4];
  int s[4];                   // s = N_l^T g0 reduced into the M_l^T box
  int w[4];                   // phase weights: phi(h) = exp(-2 pi i (w.h mod E)/E)
  int E;                      // phase modulus (largest elementary divisor of M_l)
  const float2* tw;           // exp(-2 pi i t / E), t in [0, E)
  // 32-bit index path (every intermediate of the fiber maps below 2^30 in
  // magnitude, checked on the host): divisions by the box diagonals and by E
  // through FastDiv
  int narrow;
  FastDiv fKN[4], fHM[4], fE;
};

// Consecutive levels l .. l+K-1 of the q = 2 split run as one launch: a
// thread owns one fiber of the coarsest level and the tree of 2^K - 1 fibers
// below it, so the low-pass data between the levels stays in registers.
constexpr int kMaxChain = 4;

struct SplitChain {
  SplitDesc sd[kMaxChain];          // levels l .. l+K-1 (every one on the 32-bit path)
  const float* mask[kMaxChain];     // scaling masks, natural G(M_j^T)
  float2* d2[kMaxChain];            // wavelet channel of every level, natural G(N_j^T)
  long long d2_bs[kMaxChain];       // batch strides of d2
};

// One level of the q-channel split, q = |det J| > 2 (natural orders).  The
// fiber of k in G(N_l^T) is h_l = k + N_l^T g_l reduced into the Hermite box
// of M_l^T, g_0 = 0, g_1 .. g_{q-1} the other classes of G(J^T) in the natural
// order of the Hermite box of J^T.
constexpr int kMaxQ = 16;

struct SplitQDesc {
  long long mM;               // |det M_l|
  long long mN;               // |det N_l| = mM / q
  int d;
  int q;
  int KN[4];                  // natural box of N_l^T (Hermite diagonal)
  int HM[4][4];               // column Hermite form of M_l^T
  long long hstride[4];
  int s[kMaxQ][4];            // N_l^T g_l reduced into the M_l^T box (s[0] = 0)
  float rsq;                  // 1 / sqrt(q)
  int narrow;                 // 32-bit index path (bounds checked on the host)
  FastDiv fKN[4], fHM[4];
};

}  // namespace lfft
