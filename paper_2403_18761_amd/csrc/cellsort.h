// Counting sort of points into the cells of a grid, in Morton order (internal).
#pragma once

#include <hip/hip_runtime.h>

#include "rpd_common.h"
#include "rpd_launch.h"

namespace rpd {

// float -> unsigned with the same order (negative values included)
__device__ inline unsigned order_bits(float f) {
  const unsigned b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float from_order_bits(unsigned k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The cells are those of a 64^3 grid over the points' box, or, with directions, of a 32^3 grid for each of the six
// dominant axes of a point's direction. Runs are at most len consecutive points of one coarse cell (64 cells), so that
// no run spans a jump of the Morton curve: a few runs as wide as the whole set took longer than all others together.
struct CellSort {
  unsigned* box;   // [6] the points' box as order-preserving bits: low corner, complement of the high corner
  int* n_runs;
  int* tiles;      // per tile of cells, the first position
  int* cells;      // per cell, the first position within its tile
  int* order;      // [n] the points' indices by cell (any order within a cell)
  int* rank;       // [n] a point's number in its cell
  int2* runs;      // [cell_sort_runs(n, len)] first position and number; the first n_runs of them are in use
};
size_t cell_sort_runs(long long n, int len);
size_t cell_sort_bytes(long long n, int len);
CellSort cell_sort_layout(void* memory, long long n, int len);  // memory 8-byte aligned
// The sum of cnt over a kernel's workgroups (below 2^20, 64 of them, every thread of each calls this), from the last one to
// arrive, in out and, if not null, in host (pinned memory). total must be zero before.
__device__ inline void probe_total(int cnt, int* total, int* out, int* host) {
  __shared__ int s_sum;
  if (threadIdx.x == 0) s_sum = 0;
  __syncthreads();
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
  if ((threadIdx.x & 63) == 0 && cnt) atomicAdd(&s_sum, cnt);
  __syncthreads();
  if (threadIdx.x) return;
  const int old = atomicAdd(total, (1 << 20) + s_sum);
  if (old >> 20 != (int)gridDim.x - 1) return;
  const int sum = (old & ((1 << 20) - 1)) + s_sum;
  *out = sum;
  if (host) *host = sum;
}

// In three steps, with the caller's other work between them: the jobs that clear what a sort counts in, the points' box,
// and the rest. Point k is the mean of npt vectors (3 floats each) at pts + stride k; dirs: null, or 3 floats per point.
void cell_sort_clear(FillList& L, const CellSort& S);
hipError_t launch_cell_box(const float* pts, int stride, int npt, int n, const CellSort& S, hipStream_t s);
hipError_t launch_cell_sort(const float* pts, int stride, int npt, const float* dirs, int n, int len,
                            const CellSort& S, hipStream_t s);

}  // namespace rpd
