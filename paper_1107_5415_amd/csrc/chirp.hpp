// Shapes of the chirp-z kernels, shared by the planner and chirp.hip.
#pragma once
#include <hip/hip_runtime.h>

namespace lfft {

constexpr int chirp_high_bit(int i) { return i < 2 ? i : 2 * chirp_high_bit(i / 2); }

// pencils (rows) per workgroup of an N-point convolution: 2048 points
__host__ __device__ constexpr int chirp_width(int N) { return N >= 2048 ? 1 : 2048 / N; }
// columns per workgroup of a long axis with H rows: 64-byte segments, and
// 2048 points for the shortest columns
__host__ __device__ constexpr int chirp_col_width(int H) { return H >= 256 ? 8 : 2048 / H; }
// rows H of a long axis's convolution of N = H R points (2^15 <= N <= 2^24):
// short columns while the rows stay below 2048 points, so that 10^5-point
// axes still give every CU a workgroup of 2048 points; R <= 16384
__host__ __device__ constexpr int chirp_rows_of(int N) {
  return N <= 32768 ? 128 : N <= 262144 ? 256 : N <= 1048576 ? 512 : 1024;
}

}  // namespace lfft
