// Medial spheres by sphere shrinking (Sec. 5.1, Fig. tech_sphere_gen (a)): the maximal ball that is tangent to the
// surface at a pin point p (inward unit normal n) and contains no surface point in its interior.
//
// The shrinking iteration replaces the radius by the radius of the ball through p and the surface point nearest to
// the current centre until the ball is empty; its fixed point is known in closed form. A surface point q lies strictly
// inside the ball of centre p + r n and radius r iff r > rho(q) = |q - p|^2 / (2 n.(q - p)) (for n.(q - p) > 0), so the
// maximal empty ball has radius r* = min over surface points q of rho(q). Over one triangle the smallest rho is
// reached where the growing ball first touches it: at a vertex, at a stationary point of rho along an edge (a
// quadratic in the edge parameter), or at the point where the ball is tangent to the triangle's plane (if that point
// lies in the triangle). So no iteration and no nearest-point search is needed: the result is that minimum over every
// surface triangle. Few (pin, triangle) pairs: brute force. Many: pins and triangles are sorted into grid cells, and
// 64 neighbouring pins with about the same normal evaluate only the triangles whose bounding sphere a ball smaller
// than the least radius so far can touch (k_shrink_near), where a few probes say that this leaves out enough of them.
// Both evaluate a triangle with the same expressions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "rpd.h"
#include "rpd_host.h"
#include "cellsort.h"
#include "rpd_launch.h"

namespace rpd {
namespace {

constexpr int SHR_THREADS = 256;
constexpr int SHR_R = 2;  // pins per thread

// rho at q = p + w (w = q - p): |w|^2 / (2 n.w) where n.w > 0, else +inf
__device__ inline float rho_of(float wx, float wy, float wz, float nx, float ny, float nz) {
  const float l = nx * wx + ny * wy + nz * wz;
  return l > 0.f ? (wx * wx + wy * wy + wz * wz) / (2.f * l) : INFINITY;
}

// smallest rho along the edge a + s e, s in (0, 1): stationary points of |w + s e|^2 / (2 (alpha + beta s)),
// roots of A beta s^2 + 2 A alpha s + (2 B alpha - C beta) = 0 with A = e.e, B = w.e, C = w.w
__device__ inline float edge_rho(float wx, float wy, float wz, float ex, float ey, float ez, float nx, float ny,
                                 float nz) {
  const float A = ex * ex + ey * ey + ez * ez, B = wx * ex + wy * ey + wz * ez, C = wx * wx + wy * wy + wz * wz;
  const float al = nx * wx + ny * wy + nz * wz, be = nx * ex + ny * ey + nz * ez;
  float best = INFINITY;
  auto take = [&](float s) {
    if (s > 0.f && s < 1.f) {
      const float L = al + be * s;
      if (L > 0.f) best = fminf(best, (C + s * (2.f * B + s * A)) / (2.f * L));
    }
  };
  const float qa = A * be, qb = 2.f * A * al, qc = 2.f * B * al - C * be;
  if (fabsf(qa) > 1e-30f) {
    const float disc = qb * qb - 4.f * qa * qc;
    if (disc >= 0.f) {
      const float sd = __builtin_amdgcn_sqrtf(disc);
      take((-qb + sd) / (2.f * qa));
      take((-qb - sd) / (2.f * qa));
    }
  } else if (fabsf(qb) > 1e-30f) {
    take(-qc / qb);
  }
  return best;
}

// a triangle's bounding sphere (not finite, or too large for its squares: NaN, never passed over)
__device__ inline float4 triangle_bound(const float* v) {
  const float c[3] = {(v[0] + v[3] + v[6]) * (1.f / 3.f), (v[1] + v[4] + v[7]) * (1.f / 3.f),
                      (v[2] + v[5] + v[8]) * (1.f / 3.f)};
  float d2 = 0.f;
  for (int k = 0; k < 3; ++k) {
    const float x = v[3 * k] - c[0], y = v[3 * k + 1] - c[1], z = v[3 * k + 2] - c[2];
    d2 = fmaxf(d2, x * x + y * y + z * z);
  }
  return isfinite(d2) && isfinite(c[0] + c[1] + c[2]) ? make_float4(c[0], c[1], c[2], sqrtf(d2) * 1.0001f)
                                                      : make_float4(NAN, NAN, NAN, NAN);
}

// triangle records: (a, 0) (e1 = b - a, 0) (e2 = c - a, 0) (unit normal m, 0) (dual basis u1 of e1, e2) (u2), as six
// float4, in FP64 then rounded; u1.e1 = 1, u1.e2 = 0 and u2 the other way round give barycentric coordinates
// (SORTED: record k is of triangle order[k], and bound[k] its bounding sphere; else of triangle k)
template <bool SORTED>
__global__ void k_shrink_prep(const float* tri, long long nt, const int* order, float4* rec, float4* bound) {
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < nt; t += (long long)gridDim.x * blockDim.x) {
    const float* v = tri + 9 * (SORTED ? (long long)order[t] : t);
    if (SORTED) bound[t] = triangle_bound(v);
    const double ax = v[0], ay = v[1], az = v[2];
    const double e1x = v[3] - ax, e1y = v[4] - ay, e1z = v[5] - az;
    const double e2x = v[6] - ax, e2y = v[7] - ay, e2z = v[8] - az;
    double mx = e1y * e2z - e1z * e2y, my = e1z * e2x - e1x * e2z, mz = e1x * e2y - e1y * e2x;
    const double mm = sqrt(mx * mx + my * my + mz * mz);
    const double g11 = e1x * e1x + e1y * e1y + e1z * e1z, g12 = e1x * e2x + e1y * e2y + e1z * e2z,
                 g22 = e2x * e2x + e2y * e2y + e2z * e2z;
    const double det = g11 * g22 - g12 * g12;
    float4* R = rec + 6 * t;
    R[0] = make_float4(v[0], v[1], v[2], 0.f);
    R[1] = make_float4((float)e1x, (float)e1y, (float)e1z, 0.f);
    R[2] = make_float4((float)e2x, (float)e2y, (float)e2z, 0.f);
    if (mm > 0.0 && det > 0.0) {
      mx /= mm;
      my /= mm;
      mz /= mm;
      const double i11 = g22 / det, i12 = -g12 / det, i22 = g11 / det;
      R[3] = make_float4((float)mx, (float)my, (float)mz, 1.f);
      R[4] = make_float4((float)(i11 * e1x + i12 * e2x), (float)(i11 * e1y + i12 * e2y), (float)(i11 * e1z + i12 * e2z),
                         0.f);
      R[5] = make_float4((float)(i12 * e1x + i22 * e2x), (float)(i12 * e1y + i22 * e2y), (float)(i12 * e1z + i22 * e2z),
                         0.f);
    } else {  // degenerate triangle: vertices and edges only
      R[3] = make_float4(0.f, 0.f, 0.f, 0.f);
      R[4] = make_float4(0.f, 0.f, 0.f, 0.f);
      R[5] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
}

// the smallest rho over one triangle (its record) for the pin p with normal n
// (by value: with references the brute-force loop got 16 instructions more)
__device__ __forceinline__ float triangle_rho(float4 A, float4 E1, float4 E2, float4 M, float4 U1, float4 U2, float px,
                                              float py, float pz, float nx, float ny, float nz) {
  // vertices
  const float wx = A.x - px, wy = A.y - py, wz = A.z - pz;
  float v = rho_of(wx, wy, wz, nx, ny, nz);
  v = fminf(v, rho_of(wx + E1.x, wy + E1.y, wz + E1.z, nx, ny, nz));
  v = fminf(v, rho_of(wx + E2.x, wy + E2.y, wz + E2.z, nx, ny, nz));
  // edges a->b, a->c, b->c
  v = fminf(v, edge_rho(wx, wy, wz, E1.x, E1.y, E1.z, nx, ny, nz));
  v = fminf(v, edge_rho(wx, wy, wz, E2.x, E2.y, E2.z, nx, ny, nz));
  v = fminf(v, edge_rho(wx + E1.x, wy + E1.y, wz + E1.z, E2.x - E1.x, E2.y - E1.y, E2.z - E1.z, nx, ny, nz));
  // tangency to the plane m.x = m.a at a point of the triangle: |m.(p + r n) - m.a| = r
  if (M.w != 0.f) {
    const float dl = -(M.x * wx + M.y * wy + M.z * wz);  // m.(p - a)
    const float mu = M.x * nx + M.y * ny + M.z * nz;
    for (int sg = 0; sg < 2; ++sg) {
      const float den = sg ? -(1.f + mu) : (1.f - mu);
      const float rr = dl / den;
      if (den != 0.f && rr > 0.f) {
        // tangent point relative to a: p + rr n - (m.(p + rr n - a)) m - a
        const float h = dl + rr * mu;
        const float tx = -wx + rr * nx - h * M.x, ty = -wy + rr * ny - h * M.y, tz = -wz + rr * nz - h * M.z;
        const float b1 = U1.x * tx + U1.y * ty + U1.z * tz, b2 = U2.x * tx + U2.y * ty + U2.z * tz;
        if (b1 >= 0.f && b2 >= 0.f && b1 + b2 <= 1.f) v = fminf(v, rr);
      }
    }
  }
  return v;
}

__global__ __launch_bounds__(SHR_THREADS) void k_shrink(const float4* __restrict__ rec, long long nt,
                                                        const float* __restrict__ pin, const float* __restrict__ nrm,
                                                        const int* __restrict__ own, long long n,
                                                        unsigned* __restrict__ best_bits) {
  const int chunks = gridDim.y, c = blockIdx.y;
  const long long base = (long long)blockIdx.x * (SHR_THREADS * SHR_R) + threadIdx.x;
  float px[SHR_R], py[SHR_R], pz[SHR_R], nx[SHR_R], ny[SHR_R], nz[SHR_R], best[SHR_R];
  long long skip[SHR_R];
  for (int r = 0; r < SHR_R; ++r) {
    const long long s = base + (long long)r * SHR_THREADS;
    const long long sc = s < n ? s : n - 1;
    px[r] = pin[3 * sc];
    py[r] = pin[3 * sc + 1];
    pz[r] = pin[3 * sc + 2];
    nx[r] = nrm[3 * sc];
    ny[r] = nrm[3 * sc + 1];
    nz[r] = nrm[3 * sc + 2];
    skip[r] = own ? own[sc] : -1;
    best[r] = INFINITY;
  }
  const long long t0 = nt * c / chunks, t1 = nt * (c + 1) / chunks;
  for (long long t = t0; t < t1; ++t) {
    const float4* R = rec + 6 * t;
    const float4 A = R[0], E1 = R[1], E2 = R[2], M = R[3], U1 = R[4], U2 = R[5];
    for (int r = 0; r < SHR_R; ++r) {
      const float v = triangle_rho(A, E1, E2, M, U1, U2, px[r], py[r], pz[r], nx[r], ny[r], nz[r]);
      if (t != skip[r]) best[r] = fminf(best[r], v);
    }
  }
  for (int r = 0; r < SHR_R; ++r) {
    const long long s = base + (long long)r * SHR_THREADS;
    if (s < n && best[r] < INFINITY) atomicMin(&best_bits[s], __float_as_uint(best[r]));  // positive floats
  }
}

// bounding spheres of SHR_CLUSTER consecutive triangles
constexpr int SHR_CLUSTER = 16;
__global__ void k_shrink_clusters(const float4* bound, int nt, float4* cluster) {
  const int nc = (nt + SHR_CLUSTER - 1) / SHR_CLUSTER;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x) {
    const int k0 = c * SHR_CLUSTER, k1 = min(nt, k0 + SHR_CLUSTER);
    float m[3] = {0.f, 0.f, 0.f}, R = 0.f;
    for (int k = k0; k < k1; ++k) {
      m[0] += bound[k].x;
      m[1] += bound[k].y;
      m[2] += bound[k].z;
    }
    for (int q = 0; q < 3; ++q) m[q] *= 1.f / (float)(k1 - k0);
    for (int k = k0; k < k1; ++k) {  // (NaN bounds make the centre NaN)
      const float4 b = bound[k];
      const float x = b.x - m[0], y = b.y - m[1], z = b.z - m[2];
      R = fmaxf(R, sqrtf(x * x + y * y + z * z) + b.w);
    }
    cluster[c] = make_float4(m[0], m[1], m[2], R * 1.0001f);
  }
}

// One workgroup per run of up to 64 pins, a lane per pin; its wavefronts share the clusters of triangles. The ball of
// radius r tangent at p meets the sphere (m, R) only if |p + r n - m| <= r + R, that is 2 r (n.(m - p) + R) >=
// |m - p|^2 - R^2; so triangles (and clusters) for which this fails at the least radius so far, for every pin of the
// wavefront, are passed over. That radius starts from one vertex of every cluster. The margins cover the rounding of
// the bound and of rho near a pin. Normals of another length: rho at a
// point of the sphere is at least (|m - p| - R)^2 / (2 (n.(m - p) + R |n|)), and where the ball touches a plane in the
// sphere, |m - p|^2 - R^2 <= 2 r (n.(m - p) + R) + r^2 (1 - |n|^2).
constexpr int SHR_NEAR = 512;  // threads
__global__ __launch_bounds__(SHR_NEAR) void k_shrink_near(const float4* __restrict__ rec,
                                                          const float4* __restrict__ bound,
                                                          const float4* __restrict__ cluster,
                                                          const int* __restrict__ tri_id, int nt,
                                                          const float* __restrict__ pin, const float* __restrict__ nrm,
                                                          const int* __restrict__ own, CellSort S,
                                                          float4* __restrict__ out) {
  __shared__ unsigned s_best[64];
  if ((int)blockIdx.x >= *S.n_runs) return;
  const int2 run = S.runs[blockIdx.x];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int W = SHR_NEAR / 64;
  const int s = S.order[run.x + min(lane, run.y - 1)];
  const float px = pin[3 * (size_t)s], py = pin[3 * (size_t)s + 1], pz = pin[3 * (size_t)s + 2];
  const float nx = nrm[3 * (size_t)s], ny = nrm[3 * (size_t)s + 1], nz = nrm[3 * (size_t)s + 2];
  const int skip = own ? own[s] : -1;
  const float nn = nx * nx + ny * ny + nz * nz;
  const bool unit = fabsf(nn - 1.f) <= 1e-5f;
  if (threadIdx.x < 64) s_best[threadIdx.x] = __float_as_uint(INFINITY);
  __syncthreads();
  const int nc = (nt + SHR_CLUSTER - 1) / SHR_CLUSTER;
  float best = INFINITY;
  for (int c = w; c < nc; c += W) {
    const float4 A = rec[6 * (size_t)(c * SHR_CLUSTER)];
    const float v = rho_of(A.x - px, A.y - py, A.z - pz, nx, ny, nz);
    if (tri_id[c * SHR_CLUSTER] != skip) best = fminf(best, v);
  }
  atomicMin(&s_best[lane], __float_as_uint(best));  // positive floats
  __syncthreads();
  auto reach = [&](const float4& b) {  // (NaN: kept)
    const float x = b.x - px, y = b.y - py, z = b.z - pz;
    const float ww = x * x + y * y + z * z, l = nx * x + ny * y + nz * z;
    const float e = 1e-4f * (fabsf(x) + fabsf(y) + fabsf(z) + b.w);
    if (unit) {
      const float d = l + b.w + e;
      return !(d <= 0.f || ww * 0.999f - b.w * b.w > 2.0002f * best * d);
    }
    const float nl = sqrtf(nn), D = sqrtf(ww) * 0.999f - b.w, d = l + (b.w + e) * nl;
    const bool no_point = d <= 0.f || (D > 0.f && D * D > 2.0002f * best * d);
    const bool no_plane = ww * 0.999f - b.w * b.w > 2.0002f * best * fmaxf(l + b.w + e * fmaxf(1.f, nl), 0.f) +
                                                        1.0002f * best * best * fmaxf(1.00001f - nn, 0.f);
    return !(no_point && no_plane);
  };
  for (int c = w; c < nc; c += W) {
    best = fminf(best, __uint_as_float(s_best[lane]));
    if (!__any(reach(cluster[c]))) continue;
    const int k1 = min(nt, (c + 1) * SHR_CLUSTER);
    const float before = best;
    for (int k = c * SHR_CLUSTER; k < k1; ++k) {
      if (!__any(reach(bound[k]))) continue;
      const float4* R = rec + 6 * (size_t)k;
      const float v = triangle_rho(R[0], R[1], R[2], R[3], R[4], R[5], px, py, pz, nx, ny, nz);
      if (tri_id[k] != skip) best = fminf(best, v);
    }
    if (best < before) atomicMin(&s_best[lane], __float_as_uint(best));
  }
  __syncthreads();
  if (threadIdx.x < run.y) {
    const float r = __uint_as_float(s_best[lane]);
    out[s] = make_float4(px + r * nx, py + r * ny, pz + r * nz, r);
  }
}

// How much the culling will leave: per probe, a pin, the least rho of the triangles' vertices and the number of triangles
// whose bounding sphere a ball of that radius meets, summed over the probes, each over every stride-th triangle.
constexpr int SHR_PROBES = 64, PROBE_NT = 1024, PROBE_TRIANGLES = 4096;
__global__ __launch_bounds__(PROBE_NT) void k_shrink_probe(const float* __restrict__ tri, int nt, int stride,
                                                           const float* __restrict__ pin, const float* __restrict__ nrm,
                                                           const int* __restrict__ own, int n, int* reached, int* host) {
  __shared__ float s_min[PROBE_NT / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const long long s = (2ll * blockIdx.x + 1) * n / (2 * SHR_PROBES);
  const float px = pin[3 * s], py = pin[3 * s + 1], pz = pin[3 * s + 2];
  const float nx = nrm[3 * s], ny = nrm[3 * s + 1], nz = nrm[3 * s + 2];
  const int skip = own ? own[s] : -1;
  float best = INFINITY;
  for (int t = tid * stride; t < nt; t += PROBE_NT * stride) {
    if (t == skip) continue;
    const float* v = tri + 9 * (size_t)t;
    for (int k = 0; k < 3; ++k)
      best = fminf(best, rho_of(v[3 * k] - px, v[3 * k + 1] - py, v[3 * k + 2] - pz, nx, ny, nz));
  }
  for (int off = 32; off > 0; off >>= 1) best = fminf(best, __shfl_xor(best, off));
  if (lane == 0) s_min[tid >> 6] = best;
  __syncthreads();
  for (int k = 0; k < PROBE_NT / 64; ++k) best = fminf(best, s_min[k]);
  int cnt = 0;
  for (int t = tid * stride; t < nt; t += PROBE_NT * stride) {
    const float4 b = triangle_bound(tri + 9 * (size_t)t);
    const float x = b.x - px - best * nx, y = b.y - py - best * ny, z = b.z - pz - best * nz;
    cnt += !(sqrtf(x * x + y * y + z * z) > best + b.w) ? 1 : 0;
  }
  probe_total(cnt, reached, reached + 1, host);
}

__global__ void k_shrink_finish(const unsigned* bits, const float* pin, const float* nrm, long long n, float4* out) {
  for (long long s = blockIdx.x * (long long)blockDim.x + threadIdx.x; s < n; s += (long long)gridDim.x * blockDim.x) {
    const float r = bits[s] == 0xffffffffu ? INFINITY : __uint_as_float(bits[s]);
    out[s] = make_float4(pin[3 * s] + r * nrm[3 * s], pin[3 * s + 1] + r * nrm[3 * s + 1],
                         pin[3 * s + 2] + r * nrm[3 * s + 2], r);
  }
}

}  // namespace

// Returns when the spheres are there: the workspaces, whose sorted orders the kernels index with, go back to the pool.
void shrink_spheres(const float* tri, long long nt, const float* pins, const float* normals, const int* own,
                    long long n, hipStream_t st, float4* out, bool force) {
  if (n == 0) return;
  DBuf rec(16 * 6 * (size_t)std::max<long long>(nt, 1)), bits(4 * (size_t)n), bound, cluster, ts, ps;
  EarlyInt early;
  const DrainOnExit drain{st};
  CellSort T{}, P{};
  // The sorts and the starting radii are a fixed cost that brute force passes at about 40M pairs: of the 15,384 triangles
  // of a 64^3 torus, 2,000 pins take 320 us by brute force, 4,000 take 581 us and 321 us sorted, 15,000 2,163 and 360 us.
  // Few pins on many triangles fill the chip badly (1,000 on 65k triangles: 555 us by brute force, 595 us sorted).
  bool sorted = n >= 2048 && n < (1ll << 30) && nt < (1ll << 28) && n * nt >= 40000000ll;
  if (sorted) {
    const int stride = (int)((nt + PROBE_TRIANGLES - 1) / PROBE_TRIANGLES);
    int reached = 0;
    ts.alloc(cell_sort_bytes(nt, 64));
    ps.alloc(cell_sort_bytes(n, 64));
    T = cell_sort_layout(ts.p, nt, 64);
    P = cell_sort_layout(ps.p, n, 64);
    FillList L{};
    L.add(bits.p, 0, 2, 4);
    cell_sort_clear(L, T);
    cell_sort_clear(L, P);
    hip_check(launch_fill_multi(L, st), "fill");
    hipLaunchKernelGGL(k_shrink_probe, dim3(SHR_PROBES), dim3(PROBE_NT), 0, st, tri, (int)nt, stride, pins, normals, own,
                       (int)n, bits.as<int>(), early.p());
    hip_check(hipGetLastError(), "probe");
    // (read while the triangles are sorted)
    hip_check(early.mark(st), "probe");
    hip_check(launch_cell_box(tri, 9, 3, (int)nt, T, st), "sort triangles");
    hip_check(launch_cell_sort(tri, 9, 3, nullptr, (int)nt, 64, T, st), "sort triangles");
    hip_check(early.wait(&reached), "probe");
    // The share of the triangles that the probes' balls met, and runs of a few pins where their cells are many for them
    // (about 1,300 on a surface), against brute force's full lanes and all triangles. Times sorted and by brute force,
    // and the rule's value: 64^3 torus 0.34 and 2.16 ms (0.19) for 15,000 pins, 297 and 581 us (0.62) for 4,000, 296 and
    // 485 us (0.90) for 2,700; a cylinder of strips as long as itself 1.49 and 0.79 ms (5.3) for 20,000 pins on 5,000
    // triangles, 3.9 and 0.76 ms (18) for 5,000 on 20,000; random triangles as large as the model 7.5 and 0.68 ms (7.2).
    // The probes cost the one path 12 us, the other 45 us.
    const double met = (double)reached / ((double)SHR_PROBES * (double)((nt + stride - 1) / stride));
    const double waves = (double)n / 64;
    sorted = force || (1300 + waves) / waves * (met + 0.027) < 1.0;
  }
  if (sorted) {
    const size_t nc = (size_t)(nt + SHR_CLUSTER - 1) / SHR_CLUSTER;
    bound.alloc(16 * (size_t)nt);
    cluster.alloc(16 * nc);
    hip_check(launch_cell_box(pins, 3, 1, (int)n, P, st), "sort pins");
    hip_check(launch_cell_sort(pins, 3, 1, normals, (int)n, 64, P, st), "sort pins");
    const unsigned g = (unsigned)std::min<long long>((nt + 255) / 256, 4096);
    hipLaunchKernelGGL(k_shrink_prep<true>, dim3(g), dim3(256), 0, st, tri, nt, T.order, rec.as<float4>(),
                       bound.as<float4>());
    hipLaunchKernelGGL(k_shrink_clusters, dim3((unsigned)std::min<size_t>((nc + 255) / 256, 4096)), dim3(256), 0, st,
                       bound.as<float4>(), (int)nt, cluster.as<float4>());
    hipLaunchKernelGGL(k_shrink_near, dim3((unsigned)cell_sort_runs(n, 64)), dim3(SHR_NEAR), 0, st, rec.as<float4>(),
                       bound.as<float4>(), cluster.as<float4>(), T.order, (int)nt, pins, normals, own, P, out);
    hip_check(hipGetLastError(), "shrink");
    hip_check(hipStreamSynchronize(st), "synchronize");
    return;
  }
  hip_check(launch_fill_i32(bits.as<int>(), -1, (size_t)n, st), "fill");
  if (nt > 0) {
    hipLaunchKernelGGL(k_shrink_prep<false>, dim3((unsigned)std::min<long long>((nt + 255) / 256, 4096)), dim3(256), 0,
                       st, tri, nt, (const int*)nullptr, rec.as<float4>(), (float4*)nullptr);
    const long long blocks = (n + SHR_THREADS * SHR_R - 1) / (SHR_THREADS * SHR_R);
    long long chunks = std::max<long long>(1, std::min<long long>((2048 + blocks - 1) / blocks, nt / 32));
    chunks = std::min<long long>(chunks, 65535);
    hipLaunchKernelGGL(k_shrink, dim3((unsigned)blocks, (unsigned)chunks), dim3(SHR_THREADS), 0, st, rec.as<float4>(),
                       nt, pins, normals, own, n, bits.as<unsigned>());
    hip_check(hipGetLastError(), "shrink");
  }
  hipLaunchKernelGGL(k_shrink_finish, dim3((unsigned)std::min<long long>((n + 255) / 256, 4096)), dim3(256), 0, st,
                     bits.as<unsigned>(), pins, normals, n, out);
  hip_check(hipGetLastError(), "shrink finish");
  hip_check(hipStreamSynchronize(st), "synchronize");
}

}  // namespace rpd

extern "C" rpd_status rpd_shrink_spheres(const float* tris, int64_t n_tris, const float* pins, const float* normals,
                                         const int32_t* own_tri, int64_t n_pins, uint32_t flags, void* stream,
                                         float* spheres) {
  try {
    rpd::set_error("");
    if (n_tris < 0 || n_pins < 0) throw rpd::Failure{RPD_E_INVALID, "negative count"};
    if ((n_tris && !tris) || (n_pins && (!pins || !normals || !spheres)))
      throw rpd::Failure{RPD_E_INVALID, "null array"};
    if (n_pins == 0) return RPD_OK;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) throw rpd::Failure{RPD_E_DEVICE, "no HIP device"};
    hipStream_t st = (hipStream_t)stream;
    const bool dev = (flags & RPD_DEVICE_PTRS) != 0;
    if (dev) {
      rpd::shrink_spheres(tris, n_tris, pins, normals, own_tri, n_pins, st, (float4*)spheres,
                          (flags & RPD_FORCE_CULLING) != 0);
    } else {
      rpd::DBuf t(36 * (size_t)n_tris), p(12 * (size_t)n_pins), q(12 * (size_t)n_pins), o(4 * (size_t)n_pins),
          out(16 * (size_t)n_pins);
      const rpd::DrainOnExit drain{st};
      if (n_tris) rpd::hip_check(hipMemcpyAsync(t.p, tris, 36 * (size_t)n_tris, hipMemcpyHostToDevice, st), "upload");
      rpd::hip_check(hipMemcpyAsync(p.p, pins, 12 * (size_t)n_pins, hipMemcpyHostToDevice, st), "upload");
      rpd::hip_check(hipMemcpyAsync(q.p, normals, 12 * (size_t)n_pins, hipMemcpyHostToDevice, st), "upload");
      if (own_tri)
        rpd::hip_check(hipMemcpyAsync(o.p, own_tri, 4 * (size_t)n_pins, hipMemcpyHostToDevice, st), "upload");
      rpd::shrink_spheres(t.as<float>(), n_tris, p.as<float>(), q.as<float>(), own_tri ? o.as<int>() : nullptr, n_pins,
                          st, out.as<float4>(), (flags & RPD_FORCE_CULLING) != 0);
      rpd::hip_check(hipMemcpyAsync(spheres, out.p, 16 * (size_t)n_pins, hipMemcpyDeviceToHost, st), "download");
      rpd::hip_check(hipStreamSynchronize(st), "synchronize");
    }
    return RPD_OK;
  } catch (const rpd::Failure& f) {
    rpd::set_error(f.msg);
    return f.code;
  } catch (const std::bad_alloc&) {
    rpd::set_error("host allocation failed");
    return RPD_E_NOMEM;
  }
}
