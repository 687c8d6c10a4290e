// Distance from surface samples to the enveloping volume of a medial mesh (Sec. 4.3, geometric preservation).
//
// The enveloping volume of a medial vertex is its sphere, of an edge the medial cone (spheres interpolated linearly
// between its two end spheres) and of a triangle the medial slab (spheres interpolated over the triangle), Sec. 3.2.
// For a sample q and an element whose spheres are B(c(t), r(t)), t over a segment or a triangle, the value is
// min_t |q - c(t)| - r(t): the Euclidean distance to the element's volume when q is outside it, minus the depth
// when inside. The result per sample is the minimum over every element of the mesh, and the element reaching it.
//
// The function of t is convex, so its minimum over an element lies either at an interior stationary point or on the
// element's boundary, and the boundary of a cone (its end spheres) and of a slab (its three cones) are elements of
// the mesh themselves when the mesh lists every face of its simplices. Each element is therefore evaluated only at
// its interior stationary point, in closed form (k = slope of r along a unit cone axis, g = in-plane gradient of r
// over a slab, d = q - c_1):
//   sphere: |d| - r
//   cone:   h sqrt(1 - k^2) - k u - r_1, with u = d . axis, h = |d x axis|, valid when the stationary axial position
//           u + k h / sqrt(1 - k^2) lies in [0, L]  (|k| < 1; otherwise one end sphere contains the other)
//   slab:   |H| sqrt(1 - |g|^2) - g . d - r_1, with H = d . normal, valid when the stationary centre
//           q - H normal + g |H| / sqrt(1 - |g|^2) lies in the triangle  (|g| < 1)
// and an element whose stationary point falls outside is left to its boundary elements.
//
// Two paths. Few samples: brute force over all elements: each thread keeps four samples in registers, element records
// are read with uniform (scalar) loads, and the element lists are split into chunks over the grid's second dimension so
// that the launch fills the chip; per-sample minima meet in one 64-bit atomicMin of (order-preserving float bits,
// element id), which also breaks exact ties towards the lower element id. Many samples: the samples are sorted into the
// cells of a grid, and the wavefronts of 64 neighbouring samples evaluate only the elements whose bounding sphere
// reaches as near as the minimum can be (k_env_near), where a few probes say that this leaves out enough of them. Both
// evaluate an element with the same expressions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <optional>
#include <type_traits>

#include "rpd.h"
#include "rpd_host.h"
#include "cellsort.h"
#include "rpd_launch.h"

namespace rpd {
namespace {

constexpr int ENV_THREADS = 256;
constexpr int ENV_R = 4;  // samples per thread
constexpr int ENV_SAMPLES_PER_BLOCK = ENV_THREADS * ENV_R;
constexpr int CONE_F4 = 3, SLAB_F4 = 5;
constexpr double ENV_COND = 100.0;     // largest slope or aspect whose FP32 value k_env_near bounds

__device__ inline double3 sub3(double3 a, double3 b) { return make_double3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ inline double dot3(double3 a, double3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline double3 cross3(double3 a, double3 b) {
  return make_double3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ inline double3 c3(float4 s) { return make_double3(s.x, s.y, s.z); }
__device__ inline float4 f4(double3 v, double w) { return make_float4((float)v.x, (float)v.y, (float)v.z, (float)w); }

// element records, in FP64 then rounded: cone = (c1, r1) (axis, L) (k, sqrt(1-k^2), k / sqrt(1-k^2), 0);
// slab = (c1, r1) (normal, sqrt(1-|g|^2)) (g, s m1.g) (m1, s m2.g) (m2, 0) with s = 1 / sqrt(1 - |g|^2) and
// (m1, m2) the in-plane dual basis of the triangle's edge vectors e1 = c2 - c1, e2 = c3 - c1
// bound (or null): per element (spheres, cones, slabs) a sphere (centre, R) such that the element's value at q is at
// least |q - centre| - R: all of its interpolated spheres lie inside. R = -inf: the element has no value anywhere;
// +inf: its record is so ill-conditioned that its FP32 value may leave that bound.
__device__ inline float4 bound_of(const float4* v, int n, bool value, double cond) {
  double3 m = make_double3(0, 0, 0);
  for (int k = 0; k < n; ++k) m = make_double3(m.x + v[k].x / (double)n, m.y + v[k].y / (double)n, m.z + v[k].z / (double)n);
  const float4 b = f4(m, value ? INFINITY : -INFINITY);
  if (!value || !(cond < ENV_COND)) return b;
  double R = -INFINITY;
  for (int k = 0; k < n; ++k) {  // from the rounded centre: far from the origin it is as far off as a small element is long
    const double3 d = sub3(c3(v[k]), c3(b));
    R = fmax(R, sqrt(dot3(d, d)) + v[k].w);
  }
  return make_float4(b.x, b.y, b.z, (float)(R + 1e-6 * fabs(R)));
}

__global__ void k_env_prep(const float4* sph, int ns, const int* edges, int ne, const int* tris, int nf,
                           float4* cone, float4* slab, int* status, float4* bound) {
  if (bound)
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < ns; q += gridDim.x * blockDim.x) bound[q] = sph[q];
  const int n = ne + nf;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
    if (q < ne) {
      const int i = edges[2 * q], j = edges[2 * q + 1];
      float4* R = cone + CONE_F4 * (size_t)q;
      if (i < 0 || j < 0 || i >= ns || j >= ns) {
        atomicOr(status, ST_INVALID);
        R[0] = make_float4(0.f, 0.f, 0.f, 0.f);
        R[1] = make_float4(0.f, 0.f, 0.f, -1.f);
        R[2] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (bound) bound[ns + q] = make_float4(0.f, 0.f, 0.f, INFINITY);  // the call fails
        continue;
      }
      const float4 a = sph[i], b = sph[j];
      const double3 e = sub3(c3(b), c3(a));
      const double L = sqrt(dot3(e, e)), dr = (double)b.w - (double)a.w;
      R[0] = a;
      if (L > 0.0 && fabs(dr) < L) {
        const double k = dr / L, sq = sqrt(1.0 - k * k);
        R[1] = f4(make_double3(e.x / L, e.y / L, e.z / L), L);
        R[2] = make_float4((float)k, (float)sq, (float)(k / sq), 0.f);
        if (bound) {
          const float4 v[2] = {a, b};
          bound[ns + q] = bound_of(v, 2, true, fabs(k / sq));
        }
      } else {  // one end sphere contains the other: no interior stationary point
        R[1] = make_float4(0.f, 0.f, 0.f, -1.f);
        R[2] = make_float4(0.f, 0.f, 0.f, 0.f);
        // (t = u, in [0, -1] for no u: no value, whatever the sample; NaN inputs are left to the evaluation)
        if (bound) bound[ns + q] = make_float4(a.x, a.y, a.z, L == L && dr == dr ? -INFINITY : INFINITY);
      }
    } else {
      const int f = q - ne;
      const int i = tris[3 * f], j = tris[3 * f + 1], k = tris[3 * f + 2];
      float4* R = slab + SLAB_F4 * (size_t)f;
      const float4 inert[SLAB_F4] = {make_float4(0.f, 0.f, 0.f, -INFINITY), make_float4(0.f, 0.f, 0.f, 0.f),
                                     make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f),
                                     make_float4(0.f, 0.f, 0.f, 0.f)};  // value +inf everywhere
      if (i < 0 || j < 0 || k < 0 || i >= ns || j >= ns || k >= ns) {
        atomicOr(status, ST_INVALID);
        for (int w = 0; w < SLAB_F4; ++w) R[w] = inert[w];
        if (bound) bound[ns + q] = make_float4(0.f, 0.f, 0.f, INFINITY);  // the call fails
        continue;
      }
      const float4 a = sph[i], b = sph[j], c = sph[k];
      const double3 e1 = sub3(c3(b), c3(a)), e2 = sub3(c3(c), c3(a));
      const double g11 = dot3(e1, e1), g12 = dot3(e1, e2), g22 = dot3(e2, e2);
      const double det = g11 * g22 - g12 * g12;
      bool ok = det > 1e-12 * g11 * g22;  // sin^2 of the corner angle; thinner slabs are left to their cones
      double3 m1 = make_double3(0, 0, 0), m2 = m1, g = m1, nrm = m1;
      double gg = 1.0;
      if (ok) {
        const double i11 = g22 / det, i12 = -g12 / det, i22 = g11 / det;
        m1 = make_double3(i11 * e1.x + i12 * e2.x, i11 * e1.y + i12 * e2.y, i11 * e1.z + i12 * e2.z);
        m2 = make_double3(i12 * e1.x + i22 * e2.x, i12 * e1.y + i22 * e2.y, i12 * e1.z + i22 * e2.z);
        const double d1 = (double)b.w - (double)a.w, d2 = (double)c.w - (double)a.w;
        g = make_double3(d1 * m1.x + d2 * m2.x, d1 * m1.y + d2 * m2.y, d1 * m1.z + d2 * m2.z);
        gg = dot3(g, g);
        const double3 nc = cross3(e1, e2);
        const double nn = sqrt(dot3(nc, nc));
        nrm = make_double3(nc.x / nn, nc.y / nn, nc.z / nn);
        ok = gg < 1.0;
      }
      if (!ok) {  // degenerate triangle, or one sphere's cone contains the slab's interior: boundary only
        for (int w = 0; w < SLAB_F4; ++w) R[w] = inert[w];
        if (bound) bound[ns + q] = make_float4(a.x, a.y, a.z, INFINITY);  // (the inert record's value is +inf)
        continue;
      }
      const double sq = sqrt(1.0 - gg), s = 1.0 / sq;
      if (bound) {
        const float4 v[3] = {a, b, c};
        const double l = sqrt(fmax(fmax(g11, g22), g11 + g22 - 2.0 * g12));  // the longest edge
        bound[ns + q] = bound_of(v, 3, true, fmax(s, l * sqrt(fmax(dot3(m1, m1), dot3(m2, m2)))));
      }
      R[0] = a;
      R[1] = f4(nrm, sq);
      R[2] = f4(g, s * dot3(m1, g));
      R[3] = f4(m1, s * dot3(m2, g));
      R[4] = f4(m2, 0.0);
    }
  }
}

// running minimum of a sample; with ID the element reaching it too (strict: the lower id of a chunk keeps a tie)
template <bool ID>
__device__ inline void keep_min(float f, int id, float& best, int& best_id) {
  if (ID) {
    if (f < best) {
      best = f;
      best_id = id;
    }
  } else {
    best = fminf(best, f);
  }
}

// the value of one element at a sample (+inf where its stationary point lies outside)
__device__ __forceinline__ float value_sphere(const float4& S, float qx, float qy, float qz) {
  const float dx = qx - S.x, dy = qy - S.y, dz = qz - S.z;
  return __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz) - S.w;
}
__device__ __forceinline__ float value_cone(const float4& A, const float4& B, const float4& K, float qx, float qy,
                                            float qz) {
  const float dx = qx - A.x, dy = qy - A.y, dz = qz - A.z;
  const float u = dx * B.x + dy * B.y + dz * B.z;
  const float cx = dy * B.z - dz * B.y, cy = dz * B.x - dx * B.z, cz = dx * B.y - dy * B.x;
  const float h = __builtin_amdgcn_sqrtf(cx * cx + cy * cy + cz * cz);
  const float t = u + K.z * h;
  return (t >= 0.f && t <= B.w) ? K.y * h - K.x * u - A.w : INFINITY;
}
__device__ __forceinline__ float value_slab(const float4& A, const float4& Nn, const float4& G, const float4& M1,
                                            const float4& M2, float qx, float qy, float qz) {
  const float dx = qx - A.x, dy = qy - A.y, dz = qz - A.z;
  const float aH = fabsf(dx * Nn.x + dy * Nn.y + dz * Nn.z);
  const float gd = dx * G.x + dy * G.y + dz * G.z;
  const float al = dx * M1.x + dy * M1.y + dz * M1.z + aH * G.w;
  const float be = dx * M2.x + dy * M2.y + dz * M2.z + aH * M1.w;
  const bool in = al >= 0.f && be >= 0.f && al + be <= 1.f;
  return in ? aH * Nn.w - gd - A.w : INFINITY;
}

template <bool ID>
__global__ __launch_bounds__(ENV_THREADS) void k_env_dist(const float* __restrict__ xyz, long long n,
                                                          const float4* __restrict__ sph, int ns,
                                                          const float4* __restrict__ cone, int ne,
                                                          const float4* __restrict__ slab, int nf,
                                                          unsigned long long* __restrict__ best_key) {
  const int chunks = gridDim.y, c = blockIdx.y;
  const long long base = (long long)blockIdx.x * ENV_SAMPLES_PER_BLOCK + threadIdx.x;
  float qx[ENV_R], qy[ENV_R], qz[ENV_R], best[ENV_R];
  int bid[ENV_R];
  for (int r = 0; r < ENV_R; ++r) {
    const long long s = base + (long long)r * ENV_THREADS;
    const long long sc = s < n ? s : (n - 1);
    qx[r] = xyz[3 * sc];
    qy[r] = xyz[3 * sc + 1];
    qz[r] = xyz[3 * sc + 2];
    best[r] = INFINITY;
    bid[r] = ID ? -1 : 0;
  }
  // this chunk's share of each list (uniform bounds)
  const int s0 = (int)((long long)ns * c / chunks), s1 = (int)((long long)ns * (c + 1) / chunks);
  const int e0 = (int)((long long)ne * c / chunks), e1 = (int)((long long)ne * (c + 1) / chunks);
  const int f0 = (int)((long long)nf * c / chunks), f1 = (int)((long long)nf * (c + 1) / chunks);

  for (int p = s0; p < s1; ++p) {
    const float4 S = sph[p];
    for (int r = 0; r < ENV_R; ++r) keep_min<ID>(value_sphere(S, qx[r], qy[r], qz[r]), p, best[r], bid[r]);
  }
  for (int p = e0; p < e1; ++p) {
    const float4 A = cone[CONE_F4 * (size_t)p], B = cone[CONE_F4 * (size_t)p + 1], K = cone[CONE_F4 * (size_t)p + 2];
    for (int r = 0; r < ENV_R; ++r) keep_min<ID>(value_cone(A, B, K, qx[r], qy[r], qz[r]), ns + p, best[r], bid[r]);
  }
  for (int p = f0; p < f1; ++p) {
    const float4* R = slab + SLAB_F4 * (size_t)p;
    const float4 A = R[0], Nn = R[1], G = R[2], M1 = R[3], M2 = R[4];
    for (int r = 0; r < ENV_R; ++r)
      keep_min<ID>(value_slab(A, Nn, G, M1, M2, qx[r], qy[r], qz[r]), ns + ne + p, best[r], bid[r]);
  }
  for (int r = 0; r < ENV_R; ++r) {
    const long long s = base + (long long)r * ENV_THREADS;
    if (s < n && (ID ? bid[r] >= 0 : best[r] < INFINITY))
      atomicMin(&best_key[s], ((unsigned long long)order_bits(best[r]) << 32) | (unsigned)bid[r]);
  }
}

// The minima of 256 samples, 64 neighbouring ones per wavefront, over the elements that can hold them. An element's
// value at q is at least |q - m| - R (its bounding sphere), so at least |c - m| - rho - R for every sample within rho of
// c, and a sample's minimum is at most what it has seen so far. Per ENV_SEG elements the workgroup keeps those that
// reach the bound from its own ball, each wavefront those that reach it from the wavefront's, and evaluates them. The
// margin covers the rounding of the bounds and of the values (about ten FP32 roundings, and those of the record of an
// element of condition up to ENV_COND). 1M samples against 9,841 elements: 0.41 ms, the whole call 0.60 ms (5.8 ms by
// brute force); bound by the culling tests and FP32 evaluations that remain.
constexpr int ENV_SEG = 1024;
template <bool ID>
__global__ __launch_bounds__(256) void k_env_near(const float* __restrict__ xyz, int n, const float4* __restrict__ sph,
                                                  int ns, const float4* __restrict__ cone, int ne,
                                                  const float4* __restrict__ slab, int nf,
                                                  const float4* __restrict__ bound, CellSort srt,
                                                  float* __restrict__ dist, int* __restrict__ nearest) {
  if ((int)blockIdx.x >= *srt.n_runs) return;
  __shared__ unsigned short s_list[ENV_SEG];
  __shared__ unsigned short s_mine[4][ENV_SEG];
  __shared__ float s_red[4][8];
  __shared__ int s_n;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int2 run = srt.runs[blockIdx.x];
  const int s = srt.order[run.x + min(tid, run.y - 1)];
  const float qx = xyz[3 * (size_t)s], qy = xyz[3 * (size_t)s + 1], qz = xyz[3 * (size_t)s + 2];
  // the wavefront's and the workgroup's balls
  float lo[3] = {qx, qy, qz}, hi[3] = {qx, qy, qz};
  auto ball = [&](float* c) {  // centre of the box, radius over the box's corners
    float r2 = 0.f;
    for (int k = 0; k < 3; ++k) {
      c[k] = 0.5f * (lo[k] + hi[k]);
      const float h = fmaxf(hi[k] - c[k], c[k] - lo[k]);
      r2 += h * h;
    }
    c[3] = __builtin_amdgcn_sqrtf(r2) * 1.00001f;
  };
  for (int k = 0; k < 3; ++k)
    for (int off = 32; off > 0; off >>= 1) {
      lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
      hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
    }
  float cw[4], cg[4];
  ball(cw);
  if (lane == 0)
    for (int k = 0; k < 3; ++k) {
      s_red[w][k] = lo[k];
      s_red[w][3 + k] = hi[k];
    }
  __syncthreads();
  for (int q = 0; q < 4; ++q)
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], s_red[q][k]);
      hi[k] = fmaxf(hi[k], s_red[q][3 + k]);
    }
  ball(cg);
  auto reach = [&](const float* c, const float4& b, float ub) {  // (NaN: kept)
    const float dx = c[0] - b.x, dy = c[1] - b.y, dz = c[2] - b.z;
    const float d = __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz);
    return !(d - c[3] - b.w > ub + 1e-4f * (d + c[3] + fabsf(ub)));
  };
  // a first bound from the spheres, at the workgroup's centre
  float ub = INFINITY;
  for (int p = tid; p < ns; p += 256) {
    const float4 S = sph[p];
    const float dx = cg[0] - S.x, dy = cg[1] - S.y, dz = cg[2] - S.z;
    ub = fminf(ub, __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz) - S.w);
  }
  auto most = [&](float v, bool largest) {  // over the workgroup
    for (int off = 32; off > 0; off >>= 1) v = largest ? fmaxf(v, __shfl_xor(v, off)) : fminf(v, __shfl_xor(v, off));
    __syncthreads();
    if (lane == 0) s_red[w][6] = v;
    __syncthreads();
    for (int q = 0; q < 4; ++q) v = largest ? fmaxf(v, s_red[q][6]) : fminf(v, s_red[q][6]);
    return v;
  };
  ub = most(ub, false) + cg[3];
  float best = INFINITY;
  int bid = -1;
  auto take = [&](float f, int id) {
    if (ID) {
      if (f < best || (f == best && id < bid)) {
        best = f;
        bid = id;
      }
    } else {
      best = fminf(best, f);
    }
  };
  const int first[4] = {0, ns, ns + ne, ns + ne + nf};
  for (int kind = 0; kind < 3; ++kind)
    for (int e0 = first[kind]; e0 < first[kind + 1]; e0 += ENV_SEG) {
      const int m = min(ENV_SEG, first[kind + 1] - e0);
      if (tid == 0) s_n = 0;
      __syncthreads();
      for (int k0 = 0; k0 < m; k0 += 256) {
        const int k = k0 + tid;
        const bool keep = k < m && reach(cg, bound[e0 + min(k, m - 1)], ub);
        const unsigned long long mk = __ballot(keep);
        int pos = 0;
        if (lane == 0 && mk) pos = atomicAdd(&s_n, __popcll(mk));
        pos = __shfl(pos, 0) + __popcll(mk & ((1ull << lane) - 1ull));
        if (keep) s_list[pos] = (unsigned short)k;
      }
      __syncthreads();
      const int cnt = s_n;
      // every sample of the wavefront has a minimum of at most this
      float ubw = best;
      for (int off = 32; off > 0; off >>= 1) ubw = fmaxf(ubw, __shfl_xor(ubw, off));
      ubw = fminf(ubw, ub);
      int mine = 0;
      for (int k0 = 0; k0 < cnt; k0 += 64) {
        const int k = k0 + lane;
        const int e = s_list[min(k, cnt - 1)];
        const bool keep = k < cnt && reach(cw, bound[e0 + e], ubw);
        const unsigned long long mk = __ballot(keep);
        if (keep) s_mine[w][mine + __popcll(mk & ((1ull << lane) - 1ull))] = (unsigned short)e;
        mine += __popcll(mk);
      }
      __builtin_amdgcn_wave_barrier();
      if (w * 64 >= run.y) mine = 0;  // no samples
      // two or four elements at a time: their records (scalar loads) arrive together
      auto each = [&](auto width, auto load_value) {
        constexpr int W = decltype(width)::value;
        for (int k = 0; k < mine; k += W) {
          int id[W];
          for (int q = 0; q < W; ++q) id[q] = e0 + __builtin_amdgcn_readfirstlane((int)s_mine[w][min(k + q, mine - 1)]);
          float f[W];
          load_value(id, f);
          for (int q = 0; q < W; ++q) take(f[q], id[q]);
        }
      };
      if (kind == 0) {
        each(std::integral_constant<int, 4>{}, [&](const int* id, float* f) {
          float4 R[4];
          for (int q = 0; q < 4; ++q) R[q] = sph[id[q]];
          for (int q = 0; q < 4; ++q) f[q] = value_sphere(R[q], qx, qy, qz);
        });
      } else if (kind == 1) {
        each(std::integral_constant<int, 4>{}, [&](const int* id, float* f) {
          float4 R[4][CONE_F4];
          for (int q = 0; q < 4; ++q)
            for (int x = 0; x < CONE_F4; ++x) R[q][x] = cone[CONE_F4 * (size_t)(id[q] - ns) + x];
          for (int q = 0; q < 4; ++q) f[q] = value_cone(R[q][0], R[q][1], R[q][2], qx, qy, qz);
        });
      } else {
        each(std::integral_constant<int, 2>{}, [&](const int* id, float* f) {
          float4 R[2][SLAB_F4];
          for (int q = 0; q < 2; ++q)
            for (int x = 0; x < SLAB_F4; ++x) R[q][x] = slab[SLAB_F4 * (size_t)(id[q] - ns - ne) + x];
          for (int q = 0; q < 2; ++q) f[q] = value_slab(R[q][0], R[q][1], R[q][2], R[q][3], R[q][4], qx, qy, qz);
        });
      }
      ub = fminf(ub, most(best, true));  // (also keeps the lists until every wavefront is done with them)
    }
  if (tid < run.y) {
    dist[s] = best;
    if (ID) nearest[s] = bid;
  }
}

// How much the culling will leave: per probe, a sample, its distance to the nearest sphere and the number of elements whose
// bounding sphere comes as near as that plus twice the reach of a wavefront's samples, summed over the probes; of many
// spheres and elements, every few. The reach is the distance to the nearest other probe, scaled to the spacing of 64 of
// the n samples as in three dimensions (on a surface it is less). 10 us, a chain of a few loads.
constexpr int ENV_PROBES = 64, PROBE_NT = 1024, PROBE_SPHERES = 8192, PROBE_ELEMENTS = 4096;
__global__ __launch_bounds__(PROBE_NT) void k_env_probe(const float* __restrict__ xyz, int n,
                                                        const float4* __restrict__ bound, int ns, int ne, int sphere_step,
                                                        int step, int* reached, int* host) {
  __shared__ float s_min[PROBE_NT / 64], s_reach;
  const int tid = threadIdx.x, lane = tid & 63;
  auto probe = [&](int p, float* q) {
    const long long s = (2ll * p + 1) * n / (2 * ENV_PROBES);
    for (int k = 0; k < 3; ++k) q[k] = xyz[3 * s + k];
  };
  float q[3];
  probe(blockIdx.x, q);
  auto nearest = [&](int e) {  // (a sphere's bound is the sphere)
    const float4 b = bound[e];
    return value_sphere(b, q[0], q[1], q[2]);
  };
  float best = INFINITY;
  for (int e = tid * sphere_step; e < ns; e += PROBE_NT * sphere_step) best = fminf(best, nearest(e));
  for (int off = 32; off > 0; off >>= 1) best = fminf(best, __shfl_xor(best, off));
  if (lane == 0) s_min[tid >> 6] = best;
  if (tid < 64) {
    float o[3], d2 = INFINITY;
    probe(tid, o);
    if (tid != (int)blockIdx.x)
      d2 = (q[0] - o[0]) * (q[0] - o[0]) + (q[1] - o[1]) * (q[1] - o[1]) + (q[2] - o[2]) * (q[2] - o[2]);
    for (int off = 32; off > 0; off >>= 1) d2 = fminf(d2, __shfl_xor(d2, off));
    if (tid == 0) s_reach = 2.f * sqrtf(d2) * cbrtf(64.f * ENV_PROBES / (float)n);
  }
  __syncthreads();
  for (int k = 0; k < PROBE_NT / 64; ++k) best = fminf(best, s_min[k]);
  const float ub = best + s_reach;
  int cnt = 0;
  for (long long e = (long long)tid * step; e < ne; e += PROBE_NT * step) cnt += !(nearest((int)e) > ub) ? 1 : 0;
  probe_total(cnt, reached, reached + 1, host);
}

__global__ void k_env_finish(const unsigned long long* key, long long n, float* dist, int* nearest) {
  for (long long s = blockIdx.x * (long long)blockDim.x + threadIdx.x; s < n; s += (long long)gridDim.x * blockDim.x) {
    const unsigned long long k = key[s];
    const bool none = k == ~0ull;
    dist[s] = none ? INFINITY : from_order_bits((unsigned)(k >> 32));
    if (nearest) nearest[s] = none ? -1 : (int)(k & 0xffffffffu);
  }
}

// Working memory of one call: the element records (CONE_F4 float4 per edge, SLAB_F4 per triangle), the per-sample
// minima (one 64-bit key per sample), and a status word with the probes' counts behind it.
constexpr int STATUS_INTS = 3;
size_t record_bytes(long long ne, long long nf) { return 16 * ((size_t)CONE_F4 * ne + (size_t)SLAB_F4 * nf); }

// Whether the samples may be sorted and the elements culled (k_env_near), and the working memory of that.
bool sorted_path(long long n, long long elements) {
  // More launches and a sort of the samples, against fewer evaluations: at 2,398
  // elements 100k samples take 180 us sorted and 213 us not, 30k samples 153 and 107 us; at 451 elements 1M samples
  // 265 and 327 us, 300k samples 162 and 138 us; at 9,841 elements 30k samples 305 and 262 us, 100k 337 and 733 us.
  return n >= 50000 && n < (1ll << 30) && elements < (1ll << 30) && n * elements >= 200000000ll;
}
// ... and whether they are, by the share of the elements that the probes reached. A wavefront's samples are those of a
// coarse cell, which fill few lanes where the cells are many for the samples, and it costs the share of the elements and
// the tests of all; brute force fills the lanes and costs all elements. Times sorted and by brute force, and the rule's
// value: surface samples and a medial mesh 0.61 and 5.8 ms (0.16) at 1M x 9,828, 337 and 425 us (0.93) at 60k x 9,445;
// elements as long as the model and samples in its volume 1.03 and 1.37 ms (0.84) at 1M x 2,400, 2.16 and 1.64 ms (1.23)
// at 300k x 9,000, 642 and 193 us (2.7) at 100k x 2,400; elements close together, far from the samples 1.93 and 1.37 ms
// (1.43) at 1M x 2,400. The probes cost the one path about 5 us, the other 40 us.
bool culling_pays(long long n, double reached) {
  const double waves = (double)n / 64;
  return (4096 + waves) / waves * (1.8 * reached + 0.1) < 1.0;
}
size_t sorted_bytes(long long n, long long elements) {
  return 16 * (size_t)elements + cell_sort_bytes(n, 256);
}

// The launches of one call on device-resident inputs and outputs, given its working memory; ev0/ev1 (optional)
// bracket the distance kernels; early (optional) reads the probes' count, else the call waits for it; force: cull
// whatever the probes say, where the sizes allow it. No allocation and no exception: returns the first HIP error.
// work (work_bytes of it): the per-sample minima, or what the sorted path keeps instead.
hipError_t envelope_launch(const float4* sph, int ns, const int* edg, long long ne, const int* tri, long long nf,
                           const float* xyz, long long n, hipStream_t st, float4* rec, void* work, size_t work_bytes,
                           int* status, float* dist, int* nearest, hipEvent_t ev0, hipEvent_t ev1, EarlyInt* early, bool force) {
  float4* cone = rec;
  float4* slab = rec + (size_t)CONE_F4 * ne;
  const long long total = ns + ne + nf;
  bool sorted = sorted_path(n, total) && sorted_bytes(n, total) <= work_bytes;
  float4* bound = sorted ? (float4*)work : nullptr;
  const CellSort S = cell_sort_layout((unsigned char*)work + 16 * (size_t)total, n, 256);
  FillList L{};
  L.add(status, 0, STATUS_INTS, 4);
  if (sorted) cell_sort_clear(L, S);
  hipError_t e = launch_fill_multi(L, st);
  if (e != hipSuccess) return e;
  if (sorted || ne + nf > 0) {
    const int g = (int)std::min<long long>((std::max<long long>(ne + nf, sorted ? ns : 0) + 255) / 256, 4096);
    hipLaunchKernelGGL(k_env_prep, dim3(g), dim3(256), 0, st, sph, ns, edg, (int)ne, tri, (int)nf, cone, slab, status,
                       bound);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (sorted) {
    const int step = (int)((total + PROBE_ELEMENTS - 1) / PROBE_ELEMENTS), seen = (int)((total + step - 1) / step);
    hipLaunchKernelGGL(k_env_probe, dim3(ENV_PROBES), dim3(PROBE_NT), 0, st, xyz, (int)n, bound, ns, (int)total,
                       (ns + PROBE_SPHERES - 1) / PROBE_SPHERES, step, status + 1, early ? early->p() : nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // (read while the samples' box is found, where there is pinned memory to read from)
    int reached = 0;
    e = early ? early->mark(st) : hipMemcpyAsync(&reached, status + 2, sizeof(int), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && ev0) e = hipEventRecord(ev0, st);
    if (e == hipSuccess) e = launch_cell_box(xyz, 3, 1, (int)n, S, st);
    if (e == hipSuccess) e = early ? early->wait(&reached) : hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    sorted = force || culling_pays(n, (double)reached / ((double)ENV_PROBES * (double)seen));
  } else if (ev0 && (e = hipEventRecord(ev0, st)) != hipSuccess) {
    return e;
  }
  if (sorted) {
    if ((e = launch_cell_sort(xyz, 3, 1, nullptr, (int)n, 256, S, st)) != hipSuccess) return e;
    const dim3 grid((unsigned)cell_sort_runs(n, 256));
    if (nearest)
      hipLaunchKernelGGL(k_env_near<true>, grid, dim3(256), 0, st, xyz, (int)n, sph, ns, cone, (int)ne, slab, (int)nf,
                         bound, S, dist, nearest);
    else
      hipLaunchKernelGGL(k_env_near<false>, grid, dim3(256), 0, st, xyz, (int)n, sph, ns, cone, (int)ne, slab, (int)nf,
                         bound, S, dist, nearest);
    if (ev1 && (e = hipEventRecord(ev1, st)) != hipSuccess) return e;
    return hipGetLastError();
  }
  unsigned long long* key = (unsigned long long*)work;  // (over the bounds)
  if ((e = launch_fill_u64(key, ~0ull, (size_t)n, st)) != hipSuccess) return e;
  // grid: sample blocks x element chunks, about 2048 workgroups in all, each chunk at least 64 elements
  const long long sblocks = (n + ENV_SAMPLES_PER_BLOCK - 1) / ENV_SAMPLES_PER_BLOCK;
  long long chunks = std::max<long long>(1, std::min<long long>((2048 + sblocks - 1) / sblocks, total / 64));
  chunks = std::min<long long>(chunks, 65535);
  if (total > 0) {
    if (nearest)
      hipLaunchKernelGGL(k_env_dist<true>, dim3((unsigned)sblocks, (unsigned)chunks), dim3(ENV_THREADS), 0, st, xyz,
                         n, sph, ns, cone, (int)ne, slab, (int)nf, key);
    else
      hipLaunchKernelGGL(k_env_dist<false>, dim3((unsigned)sblocks, (unsigned)chunks), dim3(ENV_THREADS), 0, st, xyz,
                         n, sph, ns, cone, (int)ne, slab, (int)nf, key);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (ev1 && (e = hipEventRecord(ev1, st)) != hipSuccess) return e;
  const int g = (int)std::min<long long>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_env_finish, dim3(g), dim3(256), 0, st, key, n, dist, nearest);
  return hipGetLastError();
}

// argument checks shared by both entry points (pure: no device access); 0 when the call may proceed
rpd_status envelope_args(const float* spheres, int ns, const int* edges, long long ne, const int* tris, long long nf,
                         const float* samples, long long n, const float* dist, const char** msg) {
  *msg = "";
  if (ns < 0 || ne < 0 || nf < 0 || n < 0) return *msg = "negative count", RPD_E_INVALID;
  if (ns + ne + nf > (long long)INT32_MAX) return *msg = "more than 2^31 elements", RPD_E_INVALID;
  if ((ns && !spheres) || (ne && !edges) || (nf && !tris) || (n && (!samples || !dist)))
    return *msg = "null array", RPD_E_INVALID;
  if ((n + ENV_SAMPLES_PER_BLOCK - 1) / ENV_SAMPLES_PER_BLOCK > INT32_MAX) return *msg = "too many samples", RPD_E_INVALID;
  return RPD_OK;
}

void envelope_distance(const float* spheres, int ns, const int* edges, long long ne, const int* tris, long long nf,
                       const float* samples, long long n, unsigned flags, hipStream_t st, float* dist, int* nearest,
                       float* kernel_ms) {
  const char* msg = "";
  if (rpd_status c = envelope_args(spheres, ns, edges, ne, tris, nf, samples, n, dist, &msg)) throw Failure{c, msg};
  if (n == 0) return;
  const bool dev = (flags & RPD_DEVICE_PTRS) != 0;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) throw Failure{RPD_E_DEVICE, "no HIP device"};

  DBuf d_sph, d_edge, d_tri, d_xyz, d_out, d_near, rec, work, status;
  std::optional<EarlyInt> early;
  if (sorted_path(n, ns + ne + nf)) early.emplace();
  const DrainOnExit drain{st};
  const float4* sph = (const float4*)spheres;
  const int* edg = edges;
  const int* tri = tris;
  const float* xyz = samples;
  if (!dev) {  // stage host inputs
    d_sph.alloc(16 * (size_t)ns);
    d_edge.alloc(8 * (size_t)ne);
    d_tri.alloc(12 * (size_t)nf);
    d_xyz.alloc(12 * (size_t)n);
    if (ns) hip_check(hipMemcpyAsync(d_sph.p, spheres, 16 * (size_t)ns, hipMemcpyHostToDevice, st), "upload");
    if (ne) hip_check(hipMemcpyAsync(d_edge.p, edges, 8 * (size_t)ne, hipMemcpyHostToDevice, st), "upload");
    if (nf) hip_check(hipMemcpyAsync(d_tri.p, tris, 12 * (size_t)nf, hipMemcpyHostToDevice, st), "upload");
    hip_check(hipMemcpyAsync(d_xyz.p, samples, 12 * (size_t)n, hipMemcpyHostToDevice, st), "upload");
    sph = d_sph.as<float4>();
    edg = d_edge.as<int>();
    tri = d_tri.as<int>();
    xyz = d_xyz.as<float>();
  }
  const size_t work_bytes = std::max(8 * (size_t)n, sorted_path(n, ns + ne + nf) ? sorted_bytes(n, ns + ne + nf) : 0);
  rec.alloc(record_bytes(ne, nf));
  work.alloc(work_bytes);
  status.alloc(sizeof(int) * STATUS_INTS);
  hipEvent_t ev[2] = {nullptr, nullptr};
  struct EventGuard {
    hipEvent_t* e;
    ~EventGuard() {
      for (int k = 0; k < 2; ++k)
        if (e[k]) (void)hipEventDestroy(e[k]);
    }
  } ev_guard{ev};
  if (kernel_ms) {
    *kernel_ms = 0.f;
    for (auto& e : ev) hip_check(hipEventCreate(&e), "hipEventCreate");
  }
  float* out_d = dist;
  int* out_n = nearest;
  if (!dev) {
    d_out.alloc(4 * (size_t)n);
    if (nearest) d_near.alloc(4 * (size_t)n);
    out_d = d_out.as<float>();
    out_n = nearest ? d_near.as<int>() : nullptr;
  }
  hip_check(envelope_launch(sph, ns, edg, ne, tri, nf, xyz, n, st, rec.as<float4>(), work.p, work_bytes, status.as<int>(), out_d, out_n, ev[0],
                            ev[1], early ? &*early : nullptr, (flags & RPD_FORCE_CULLING) != 0),
            "envelope distance");
  int hst = 0;
  hip_check(hipMemcpyAsync(&hst, status.p, sizeof(int), hipMemcpyDeviceToHost, st), "download");
  if (!dev) {
    hip_check(hipMemcpyAsync(dist, out_d, 4 * (size_t)n, hipMemcpyDeviceToHost, st), "download");
    if (nearest) hip_check(hipMemcpyAsync(nearest, out_n, 4 * (size_t)n, hipMemcpyDeviceToHost, st), "download");
  }
  hip_check(hipStreamSynchronize(st), "synchronize");
  if (kernel_ms) hip_check(hipEventElapsedTime(kernel_ms, ev[0], ev[1]), "hipEventElapsedTime");
  if (hst & ST_INVALID) throw Failure{RPD_E_INVALID, "an edge or triangle names a sphere out of range"};
}

// ---------------------------------------------------------------------------------------------------------------
// The no-allocation variant's working memory: one fixed region per device, reserved with the library's code
// object and held until the process ends. Host code never passes the array itself to a kernel (its name is a host
// stand-in); it looks up the region's device address once per device and uses that.
// ---------------------------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[RPD_NOALLOC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES];  // device address of `scratch` per device (nullptr until looked up)

// the current device's address of the region (looked up on the first call on that device)
rpd_status scratch_address(void** out, const char** msg) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return *msg = "no HIP device", RPD_E_DEVICE;
  if (dev >= MAX_DEVICES) return *msg = "device index beyond the scratch table", RPD_E_DEVICE;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
      return *msg = "scratch region not available on this device", RPD_E_DEVICE;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return RPD_OK;
}

// bytes of the region one call uses: status word, per-sample minima, element records, each 256-byte aligned
size_t noalloc_bytes(long long ne, long long nf, long long n) {
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  return 256 + up(8 * (size_t)n) + up(record_bytes(ne, nf));
}
}  // namespace
}  // namespace rpd

extern "C" rpd_status rpd_envelope_distance_noalloc(const float* spheres, int32_t n_spheres, const int32_t* edges,
                                                    int64_t n_edges, const int32_t* tris, int64_t n_tris,
                                                    const float* samples, int64_t n_samples, void* stream, float* dist,
                                                    int32_t* nearest) {
  using namespace rpd;
  const char* msg = "";
  rpd_status c = envelope_args(spheres, n_spheres, edges, n_edges, tris, n_tris, samples, n_samples, dist, &msg);
  if (c == RPD_OK && noalloc_bytes(n_edges, n_tris, n_samples) > (size_t)RPD_NOALLOC_SCRATCH_BYTES) {
    c = RPD_E_NOMEM;
    msg = "the samples and elements exceed the no-allocation scratch region (RPD_NOALLOC_SCRATCH_BYTES)";
  }
  if (c != RPD_OK) {
    set_error(msg);
    return c;
  }
  set_error("");
  if (n_samples == 0) return RPD_OK;
  void* base = nullptr;
  if ((c = scratch_address(&base, &msg)) != RPD_OK) {
    set_error(msg);
    return c;
  }
  unsigned char* b = (unsigned char*)base;
  int* status = (int*)b;
  // the records right behind the status word, the rest of the region behind them
  float4* rec = (float4*)(b + 256);
  const size_t at = 256 + ((record_bytes(n_edges, n_tris) + 255) & ~(size_t)255);
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = envelope_launch((const float4*)spheres, n_spheres, edges, n_edges, tris, n_tris, samples, n_samples,
                                 st, rec, b + at, (size_t)RPD_NOALLOC_SCRATCH_BYTES - at, status, dist, nearest,
                                 nullptr, nullptr, nullptr, false);
  int hst = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&hst, status, sizeof(int), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) {
    set_error(hipGetErrorString(e));
    return RPD_E_DEVICE;
  }
  if (hst & ST_INVALID) {
    set_error("an edge or triangle names a sphere out of range");
    return RPD_E_INVALID;
  }
  return RPD_OK;
}

extern "C" rpd_status rpd_envelope_distance(const float* spheres, int32_t n_spheres, const int32_t* edges,
                                            int64_t n_edges, const int32_t* tris, int64_t n_tris,
                                            const float* samples, int64_t n_samples, uint32_t flags, void* stream,
                                            float* dist, int32_t* nearest, float* kernel_ms) {
  try {
    rpd::set_error("");
    rpd::envelope_distance(spheres, n_spheres, edges, n_edges, tris, n_tris, samples, n_samples, flags,
                           (hipStream_t)stream, dist, nearest, kernel_ms);
    return RPD_OK;
  } catch (const rpd::Failure& f) {
    rpd::set_error(f.msg);
    return f.code;
  } catch (const std::bad_alloc&) {
    rpd::set_error("host allocation failed");
    return RPD_E_NOMEM;
  }
}
