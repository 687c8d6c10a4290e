// Counting sort of points into grid cells (cellsort.h): six launches, two passes over the points. The counting pass is
// bound by one returning atomic per point (80 us per million), which also hands every point its place.
#include <algorithm>

#include <hip/hip_runtime.h>

#include "cellsort.h"
#include "rpd_launch.h"

namespace rpd {
namespace {

constexpr int CELLS = 1 << 18;
constexpr int TILE = 1024;  // cells scanned per workgroup
constexpr int TILES = CELLS / TILE;
constexpr int COARSE = 64, NCOARSE = CELLS / COARSE;

struct Points {
  const float* p;
  int stride, npt;
  const float* dirs;
  int n;
  __device__ void get(int k, float* x) const {
    const float* q = p + (size_t)stride * k;
    for (int c = 0; c < 3; ++c) x[c] = q[c];
    for (int v = 1; v < npt; ++v)
      for (int c = 0; c < 3; ++c) x[c] += q[3 * v + c];
    if (npt > 1)
      for (int c = 0; c < 3; ++c) x[c] *= 1.f / (float)npt;
  }
};

__global__ __launch_bounds__(256) void k_cell_box(Points P, CellSort S) {
  __shared__ unsigned s_b[6];
  if (threadIdx.x < 6) s_b[threadIdx.x] = ~0u;
  __syncthreads();
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int s = blockIdx.x * 256 + threadIdx.x; s < P.n; s += gridDim.x * 256) {
    float x[3];
    P.get(s, x);
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], x[k]);
      hi[k] = fmaxf(hi[k], x[k]);
    }
  }
  for (int k = 0; k < 3; ++k) {
    for (int off = 32; off > 0; off >>= 1) {
      lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
      hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
    }
    if ((threadIdx.x & 63) == 0) {
      atomicMin(&s_b[k], order_bits(lo[k]));
      atomicMin(&s_b[3 + k], ~order_bits(hi[k]));
    }
  }
  __syncthreads();
  if (threadIdx.x < 6) atomicMin(&S.box[threadIdx.x], s_b[threadIdx.x]);
}

__device__ inline unsigned spread_bits(unsigned x) {  // 6 bits -> every third bit
  x = (x | (x << 8)) & 0x300fu;
  x = (x | (x << 4)) & 0x30c3u;
  return (x | (x << 2)) & 0x9249u;
}
struct Grid {
  float o[3], scale, last;
  __device__ void load(const CellSort& S, bool dirs) {
    float ext = 0.f;
    for (int k = 0; k < 3; ++k) {
      o[k] = from_order_bits(S.box[k]);
      ext = fmaxf(ext, from_order_bits(~S.box[3 + k]) - o[k]);
    }
    last = dirs ? 31.f : 63.f;
    scale = ext > 0.f ? (last + 1.f) / ext : 0.f;
  }
  __device__ int cell(const Points& P, int k) const {
    float x[3];
    P.get(k, x);
    unsigned c = 0;
    for (int q = 0; q < 3; ++q)  // clamped (NaN and infinite coordinates too: they go somewhere)
      c |= spread_bits((unsigned)fminf(fmaxf((x[q] - o[q]) * scale, 0.f), last)) << q;
    if (P.dirs) {
      const float* d = P.dirs + 3 * (size_t)k;
      const float ax = fabsf(d[0]), ay = fabsf(d[1]), az = fabsf(d[2]);
      const int a = ax >= ay && ax >= az ? 0 : ay >= az ? 1 : 2;
      c |= (unsigned)(2 * a + (d[a] < 0.f ? 1 : 0)) << 15;
    }
    return (int)c;
  }
};

__global__ __launch_bounds__(256) void k_cell_count(Points P, CellSort S) {
  Grid g;
  g.load(S, P.dirs != nullptr);
  for (int s = blockIdx.x * 256 + threadIdx.x; s < P.n; s += gridDim.x * 256)
    S.rank[s] = atomicAdd(&S.cells[g.cell(P, s)], 1);
}

__global__ __launch_bounds__(TILE) void k_cell_scan(CellSort S) {  // the counts of a tile -> positions within it
  __shared__ int s_w[TILE / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int v = S.cells[blockIdx.x * TILE + t];
  int x = v;
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  if (lane == 63) s_w[w] = x;
  __syncthreads();
  for (int q = 0; q < w; ++q) x += s_w[q];
  S.cells[blockIdx.x * TILE + t] = x - v;
  if (t == TILE - 1) S.tiles[blockIdx.x] = x;
}

// the first position of every tile, and the runs (one workgroup, four coarse cells per thread)
__global__ __launch_bounds__(1024) void k_cell_runs(CellSort S, int len) {
  static_assert(NCOARSE == 4096 && TILES == 256 && TILE == 16 * COARSE, "four coarse cells per thread");
  __shared__ int s_base[TILES + 1];
  __shared__ int s_w[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  auto prefix = [&](int v) {  // exclusive sum over the workgroup
    int x = v;
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(x, off);
      if (lane >= off) x += y;
    }
    __syncthreads();
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    for (int q = 0; q < w; ++q) x += s_w[q];
    return x - v;
  };
  const int b = prefix(t < TILES ? S.tiles[t] : 0);
  if (t <= TILES) s_base[t] = b;
  if (t < TILES) S.tiles[t] = b;
  __syncthreads();
  int first[5], n = 0;
  for (int k = 0; k < 5; ++k) {
    const int c = 4 * t + k;  // (a tile's first cell starts where the tile does)
    first[k] = s_base[c / 16] + (c % 16 ? S.cells[c * COARSE] : 0);
  }
  for (int k = 0; k < 4; ++k) n += (first[k + 1] - first[k] + len - 1) / len;
  int at = prefix(n);
  for (int k = 0; k < 4; ++k)
    for (int p = first[k]; p < first[k + 1]; p += len) S.runs[at++] = make_int2(p, min(len, first[k + 1] - p));
  if (t == 1023) *S.n_runs = at;
}

__global__ __launch_bounds__(256) void k_cell_scatter(Points P, CellSort S) {
  Grid g;
  g.load(S, P.dirs != nullptr);
  for (int s = blockIdx.x * 256 + threadIdx.x; s < P.n; s += gridDim.x * 256) {
    const int c = g.cell(P, s);
    S.order[S.tiles[c / TILE] + S.cells[c] + S.rank[s]] = s;
  }
}

}  // namespace

size_t cell_sort_runs(long long n, int len) { return (size_t)std::min<long long>(n / len + NCOARSE, n); }
size_t cell_sort_bytes(long long n, int len) {
  return 8 * cell_sort_runs(n, len) + 4 * (2 * (size_t)n + CELLS + TILES + 8);
}
CellSort cell_sort_layout(void* memory, long long n, int len) {
  CellSort S;
  S.runs = (int2*)memory;
  S.box = (unsigned*)(S.runs + cell_sort_runs(n, len));
  S.n_runs = (int*)(S.box + 6);
  S.tiles = S.n_runs + 2;
  S.cells = S.tiles + TILES;
  S.order = S.cells + CELLS;
  S.rank = S.order + n;
  return S;
}
static unsigned point_grid(int n) { return (unsigned)std::min((n + 255) / 256, 2048); }
void cell_sort_clear(FillList& L, const CellSort& S) {
  L.add(S.box, ~0ull, 6, 4);
  L.add(S.cells, 0, CELLS, 4);
}
hipError_t launch_cell_box(const float* pts, int stride, int npt, int n, const CellSort& S, hipStream_t s) {
  const Points P{pts, stride, npt, nullptr, n};
  hipLaunchKernelGGL(k_cell_box, dim3(std::min(point_grid(n), 512u)), dim3(256), 0, s, P, S);
  return hipGetLastError();
}
hipError_t launch_cell_sort(const float* pts, int stride, int npt, const float* dirs, int n, int len,
                            const CellSort& S, hipStream_t s) {
  const Points P{pts, stride, npt, dirs, n};
  const unsigned g = point_grid(n);
  hipLaunchKernelGGL(k_cell_count, dim3(g), dim3(256), 0, s, P, S);
  hipLaunchKernelGGL(k_cell_scan, dim3(TILES), dim3(TILE), 0, s, S);
  hipLaunchKernelGGL(k_cell_runs, dim3(1), dim3(1024), 0, s, S, len);
  hipLaunchKernelGGL(k_cell_scatter, dim3(g), dim3(256), 0, s, P, S);
  return hipGetLastError();
}

}  // namespace rpd
