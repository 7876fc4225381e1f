// Batched persistent launch: the lattice FFTs of many signals on patterns of
// different M.  Every pass of every lattice is cut into tiles of T elements,
// each processed by T / 16 threads with the register-resident pass body of
// fast_tile.hpp.  The tiles of all first passes (and of lattices done in one
// pass) form phase 0, the tiles of all second passes phase 1; each phase is
// one persistent launch over eight work queues, one per XCD, that the host
// fills largest lattice first, in runs of neighbouring tiles of one lattice
// (1/128 of the phase), which share an L2.
// The kernel boundary between the phases orders the two passes of every
// lattice, so the tiles need no counters, fences or waits.
//
// A workgroup takes every n-th item of the queue of its own XCD (dispatch index
// mod 8, n workgroups there).  All items are tiles of one size, so fixed
// strides come within 1% of queue heads on 512 lattices of 2^10 .. 2^18 points
// (408 against 403 us), without the atomic, the broadcast through LDS, the
// launch that cleared the heads (a 512 x 512 picture's pyramid 118 -> 102 us)
// and a state that two calls of one plan would share.
#include <hip/hip_runtime.h>

#include <atomic>

#include "fast_tile.hpp"
#include "kernels.hpp"

namespace lfft {
namespace {
using namespace dev;

// blockDim.x = T / 16 threads (128, 256 or 512) for tiles of T elements.
// qbeg[0..8]: queue boundaries of this phase.
__global__ void __launch_bounds__(512) fft_batch_kernel(const BatchPass* __restrict__ passes,
                                                        const int2* __restrict__ items,
                                                        const int* __restrict__ qbeg,
                                                        const float2* in, float2* out,
                                                        float2* ws) {
  extern __shared__ float2 lds_raw[];
  const int tid = threadIdx.x;
  const int q = blockIdx.x & 7;
  const int end = qbeg[q + 1], step = ((int)gridDim.x + 7 - q) >> 3;
  int it = qbeg[q] + (int)(blockIdx.x >> 3);
  if (it >= end) return;
  int2 next = items[it];
  for (; it < end; it += step) {
    const int pi = __builtin_amdgcn_readfirstlane(next.x);
    const long long tile = __builtin_amdgcn_readfirstlane(next.y);
    // the next item while this one runs
    if (it + step < end) next = items[it + step];
    const BatchPass& bp = passes[pi];
    const float2* src = (bp.in_buf == 0 ? in : bp.in_buf == 1 ? out : ws) + bp.in_off;
    float2* dst = (bp.out_buf == 1 ? out : ws) + bp.out_off;
    switch (bp.variant) {
      case BATCH_ROWS_NN:
        fastk::fast_tile<16, false, false, MAP_NATURAL, MAP_NATURAL, false>(bp.pd, tile, tid, src, dst, lds_raw);
        break;
      case BATCH_ROWS_NI:
        fastk::fast_tile<16, false, false, MAP_NATURAL, MAP_IDENTITY, false>(bp.pd, tile, tid, src, dst, lds_raw);
        break;
      case BATCH_COLS_NI:
        fastk::fast_tile<16, true, false, MAP_NATURAL, MAP_IDENTITY, true>(bp.pd, tile, tid, src, dst, lds_raw);
        break;
      case BATCH_ROWS_IN:
        fastk::fast_tile<16, false, false, MAP_IDENTITY, MAP_NATURAL, false>(bp.pd, tile, tid, src, dst, lds_raw);
        break;
      default:
        fastk::fast_tile<16, true, false, MAP_IDENTITY, MAP_NATURAL, false>(bp.pd, tile, tid, src, dst, lds_raw);
        break;
    }
    // (a tile ends with a barrier after its last LDS read, so the next one
    // may write)
  }
}

std::atomic<bool> g_attr{false};

hipError_t set_attr() {
  if (g_attr.load(std::memory_order_acquire)) return hipSuccess;
  hipError_t e = hipFuncSetAttribute((const void*)fft_batch_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)batch_lds_bytes(1 << 13));
  if (e == hipSuccess) g_attr.store(true, std::memory_order_release);
  return e;
}

}  // namespace

size_t batch_lds_bytes(int tile) { return (size_t)(tile + tile / 16 + fastk::kTilePad) * sizeof(float2); }

int batch_occupancy(int tile_lg) {
  if (tile_lg < 11 || tile_lg > 13 || set_attr() != hipSuccess) return 0;
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fft_batch_kernel, 1 << (tile_lg - 4),
                                                   batch_lds_bytes(1 << tile_lg)) != hipSuccess)
    return 0;
  return nb;
}

const char* batch_kernel_name(int) { return "fft_batch_kernel"; }

hipError_t launch_batch(int tile_lg, const BatchPass* passes, const int2* items, const int* qbeg,
                        const float2* in, float2* out, float2* ws, int grid, hipStream_t s) {
  if (tile_lg < 11 || tile_lg > 13 || grid < 8) return hipErrorInvalidValue;  // every queue
  hipError_t e = set_attr();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fft_batch_kernel, dim3(grid), dim3(1 << (tile_lg - 4)),
                     batch_lds_bytes(1 << tile_lg), s, passes, items, qbeg, in, out, ws);
  return hipGetLastError();
}

}  // namespace lfft
