// Tet-Cell clipping (paper Sec. 5.2) with on-the-fly fractional Euler characteristic (Sec. 4.1.2) and the gluing
// information for connected components (Sec. 4.1.1), in two kernels.
//
// Candidate kernel: one wavefront owns up to TB spatially consecutive tets. It selects the sites that can own any
// point of the group's bounding box, then per tet the candidate sites that can own a point of the tet, sorted by power
// distance at the tet centroid, and hands every tet a run of piece slots, one per candidate.
//
// Piece kernel: 64 consecutive piece slots per wavefront, one lane per piece: the tet is clipped by the bisectors of
// all other candidates with the polytope in LDS, and the piece's cell terms and element records (faces, edges, RPVs:
// chi numerators, gluing bits, lengths) are written out. No hash table and no shared accumulator is touched here: the
// emission kernel turns the records into sums.
//
// Tets with too many candidates and pieces whose predicates stay undecided in FP64 go to the large-capacity kernel,
// which computes them with FP64 constructions and exact predicates.
#include <hip/hip_runtime.h>

#include <climits>

#include <algorithm>

#include "rpd_device.h"
#include "rpd_launch.h"

namespace rpd {

// ---------------------------------------------------------------------------------------------------------------
// the terms of one nonempty piece
// ---------------------------------------------------------------------------------------------------------------
template <typename Topo>
__device__ inline int pos_of(typename Topo::W w, int p) {
  if (Topo::plane(w, 0) == p) return 0;
  if (Topo::plane(w, 1) == p) return 1;
  if (Topo::plane(w, 2) == p) return 2;
  return -1;
}

template <typename Topo>
__device__ inline long long wv_of(typename Topo::W w, const unsigned* nu, long long L) {
  return w_vertex(Topo::plane(w, 0), Topo::plane(w, 1), Topo::plane(w, 2), nu, L);
}

// What the first pass over a piece's vertices leaves for emit_out.
template <typename CL>
struct EmitAcc {
  typedef typename CL::Real T;
  typedef typename CL::MaskT Mask;
  long long sv, se;         // vertex and edge weights
  T gx, gy, gz;             // vertex sums
  int nv;
  unsigned planes;          // planes present (Topo32: at most 32 of them)
  int nface, nedge, nrpv;   // element records of the piece (elements whose smallest site is the piece's)
  Mask edge[3], rpv;        // vertices k with such an edge at position f (k below its other end), or such an RPV
  __device__ int records() const { return nface + nedge + nrpv; }
};

// vertex pass: vertex and edge weights, the first vertex of every face (kept in the clipper's table), the records
template <typename CL>
__device__ __forceinline__ void emit_scan(CL& c, const unsigned* nu, long long L, EmitAcc<CL>& e) {
  typedef typename CL::TopoT Topo;
  typedef typename Topo::W W;
  const int i = c.env.site_i;  // batch-global site id
  e.sv = e.se = 0;
  e.gx = e.gy = e.gz = 0;
  e.nv = e.nface = e.nedge = e.nrpv = 0;
  e.planes = 0;
  e.edge[0] = e.edge[1] = e.edge[2] = e.rpv = 0;
  for (auto m = c.live; m; m &= m - 1) {
    const int k = ctz_mask(m);
    const W w = c.st.topo(k);
    const auto v = c.st.get(k);
    e.gx += v.x;
    e.gy += v.y;
    e.gz += v.z;
    ++e.nv;
    const int p0 = Topo::plane(w, 0), p1 = Topo::plane(w, 1), p2 = Topo::plane(w, 2);
    e.sv += w_vertex(p0, p1, p2, nu, L);
    bool above[3];  // the plane is a bisector against a higher site
    for (int f = 0; f < 3; ++f) {
      const int p = Topo::plane(w, f);
      above[f] = p >= 4 && c.env.cand_id(p - 4) > i;
      if (c.tab.get(p) == 0) {
        c.tab.set(p, k + 1);
        if (CL::FEW_PLANES) e.planes |= 1u << (p & 31);
        e.nface += above[f] ? 1 : 0;
      }
    }
    for (int f = 0; f < 3; ++f) {
      if (k < Topo::nb(w, f)) {
        const int f1 = f == 2 ? 0 : f + 1, f2 = f == 0 ? 2 : f - 1;
        e.se += w_edge(Topo::plane(w, f1), Topo::plane(w, f2), nu, L);
        if (above[f1] && above[f2]) {
          ++e.nedge;
          e.edge[f] |= CL::bit(k);
        }
      }
    }
    if (above[0] && above[1] && above[2]) {
      ++e.nrpv;
      e.rpv |= CL::bit(k);
    }
  }
}

// The piece's cell terms and its element records, written to slot p_slot and to records [base, base + e.records()).
// Every loop takes one item of the lane's own list per trip (an edge, an RPV, a face vertex), so that lanes whose
// pieces have different shapes stay together; a loop over plane numbers and one over the face's edges inside it kept
// one lane in five busy.
template <typename CL>
__device__ __forceinline__ void emit_out(CL& c, const ShapeDesc& sd, int tl, EmitAcc<CL>& e, int p_slot, int base,
                                         const ShapeArgs& a) {
  typedef typename CL::Real T;
  typedef typename CL::TopoT Topo;
  typedef typename Topo::W W;
  const int i = c.env.site_i;
  const unsigned* nu = sd.nu + 14 * (size_t)tl;
  const long long L = sd.L;
  const int4 tn4 = reinterpret_cast<const int4*>(sd.tn)[tl];  // face neighbours (-1: boundary), one load
  const unsigned interior = (tn4.x >= 0 ? 1u : 0u) | (tn4.y >= 0 ? 2u : 0u) | (tn4.z >= 0 ? 4u : 0u) |
                            (tn4.w >= 0 ? 8u : 0u);  // bit f: face f is shared with another tet
  auto put = [&](int r, int j, int k, int z, long long num, double len) {
    ElemRec R;
    R.j = j;
    R.k = k;
    R.z = z;
    R.p = p_slot;
    R.num = num;
    R.len = len;
    a.recs[r] = R;
  };
  auto inner = [&](int p) { return p < 4 ? (int)(interior & (1u << p)) : 0; };  // the gluing bit of an interior face
  int re = base + e.nface;
  while (e.edge[0] | e.edge[1] | e.edge[2]) {  // RPE pieces
    const int k = ctz_mask(e.edge[0] | e.edge[1] | e.edge[2]);
    const auto b = CL::bit(k);
    const int f = (e.edge[0] & b) ? 0 : (e.edge[1] & b) ? 1 : 2;
    if (f == 0) e.edge[0] &= ~b;
    else if (f == 1) e.edge[1] &= ~b;
    else e.edge[2] &= ~b;
    const W wk = c.st.topo(k);
    const int n = Topo::nb(wk, f);
    const W wn = c.st.topo(n);
    const auto C = c.st.get(k), N = c.st.get(n);
    const int pa = Topo::plane(wk, f == 2 ? 0 : f + 1), pb = Topo::plane(wk, f == 0 ? 2 : f - 1);
    const int ea = pos_of<Topo>(wn, pa), eb = pos_of<Topo>(wn, pb);
    if (ea < 0 || eb < 0) atomicOr(a.status, ST_INTERNAL);
    const int sa = c.env.cand_id(pa - 4), sb = c.env.cand_id(pb - 4);
    const T lx = N.x - C.x, ly = N.y - C.y, lz = N.z - C.z;
    const long long ev = wv_of<Topo>(wk, nu, L) + wv_of<Topo>(wn, nu, L) - L;
    // the third planes at the two ends
    const int g = inner(Topo::plane(wk, f)) | inner(Topo::plane(wn, (3 - ea - eb) & 3));
    put(re++, min(sa, sb), max(sa, sb), (REC_EDGE << REC_SHIFT) | g, ev, (double)sqrt(lx * lx + ly * ly + lz * lz));
  }
  int rq = base + e.nface + e.nedge;
  for (auto m = e.rpv; m; m &= m - 1) {  // an RPV is recorded once, from its smallest site
    const W w = c.st.topo(ctz_mask(m));
    const int s0 = c.env.cand_id(Topo::plane(w, 0) - 4), s1 = c.env.cand_id(Topo::plane(w, 1) - 4),
              s2 = c.env.cand_id(Topo::plane(w, 2) - 4);
    const int lo = min(s0, min(s1, s2)), hi = max(s0, max(s1, s2)), mid = s0 + s1 + s2 - lo - hi;
    put(rq++, lo, mid, (REC_RPV << REC_SHIFT) | hi, 1, 0.0);
  }
  const T inv_nv = T(1) / T(e.nv);
  const T ax = e.gx * inv_nv, ay = e.gy * inv_nv, az = e.gz * inv_nv;

  // ---- face cycles, by ascending plane (volume fans, face terms): one vertex per trip, the first of a face starts it
  long long sf = 0;
  int cell_glue = 0;
  T vol = 0, mx = 0, my = 0, mz = 0;
  int rf = base;
  auto next_face = [&](int p) {  // the next plane with a face, or -1
    if (CL::FEW_PLANES) {
      if (!e.planes) return -1;
      const int q = ctz_mask(e.planes);
      e.planes &= e.planes - 1;
      return q;
    }
    for (++p; p < c.np; ++p)
      if (c.tab.get(p)) return p;
    return -1;
  };
  int p = next_face(-1);
  bool start = true, felem = false;
  int r = 0, nxt = 0, acur = 0, sp = -1, steps = 0, fglue = 0;
  long long fchi = 0;
  T Rx = 0, Ry = 0, Rz = 0, Cx = 0, Cy = 0, Cz = 0;
  while (p >= 0) {
    if (start) {
      nxt = c.tab.get(p) - 1;
      c.tab.set(p, 0);
    }
    const W wn = c.st.topo(nxt);
    const auto N = c.st.get(nxt);
    const int epn = pos_of<Topo>(wn, p);
    const int ea = start ? 0 : pos_of<Topo>(wn, acur);
    if (ea < 0 || epn < 0 || steps > CL::SLOTS) {  // a broken polytope: the call fails
      atomicOr(a.status, ST_INTERNAL);
      start = true;
      steps = 0;
      if (felem && rf < base + e.nface) put(rf++, 0, 0, REC_NONE << REC_SHIFT, 0, 0.0);
      felem = false;
      p = next_face(p);
      continue;
    }
    if (start) {
      r = nxt;
      sf += (p < 4) ? (long long)nu[10 + p] : L;
      if (p < 4) cell_glue |= inner(p) ? 1 << p : 16 << p;  // glue across an interior face; boundary contact
      sp = c.env.plane_site(p);
      felem = p >= 4 && sp > i;
      fchi = L;
      fglue = 0;
      steps = 0;
      Rx = N.x;
      Ry = N.y;
      Rz = N.z;
      if (felem) fchi += wv_of<Topo>(wn, nu, L);
      acur = Topo::plane(wn, epn == 2 ? 0 : epn + 1);
      nxt = Topo::nb(wn, epn == 0 ? 2 : epn - 1);
      start = false;
    } else {
      const bool closed = nxt == r;
      if (felem) {  // the edge to nxt lies on planes {p, acur}
        fchi -= w_edge(p, acur, nu, L);
        if (!closed) fchi += wv_of<Topo>(wn, nu, L);
        fglue |= inner(acur);
      }
      if (closed) {
        if (felem && rf < base + e.nface) put(rf++, sp, -1, (REC_FACE << REC_SHIFT) | fglue, fchi, 0.0);
        felem = false;
        start = true;
        p = next_face(p);
      } else {
        if (steps > 0) {  // fan triangle (R, C, N) with the apex: a tet of the piece
          T ux = Cx - Rx, uy = Cy - Ry, uz = Cz - Rz;
          T vx = N.x - Rx, vy = N.y - Ry, vz = N.z - Rz;
          T wx = ax - Rx, wy = ay - Ry, wz = az - Rz;
          T det = ux * (vy * wz - vz * wy) - uy * (vx * wz - vz * wx) + uz * (vx * wy - vy * wx);
          T tv = fabs(det) * T(1.0 / 6.0);
          vol += tv;
          mx += tv * (Rx + Cx + N.x + ax);
          my += tv * (Ry + Cy + N.y + ay);
          mz += tv * (Rz + Cz + N.z + az);
        }
        ++steps;
        const int ec = 3 - ea - epn;
        nxt = Topo::nb(wn, ea);  // leave the vertex along {p, its third plane}: the neighbour opposite acur
        acur = Topo::plane(wn, ec & 3);
      }
    }
    Cx = N.x;
    Cy = N.y;
    Cz = N.z;
  }
  // records counted but not written (a broken polytope): nothing may read stale ones
  for (; rf < base + e.nface; ++rf) put(rf, 0, 0, REC_NONE << REC_SHIFT, 0, 0.0);
  // moments were accumulated with 4x the centroid sum; shift to absolute coordinates
  const float4 o = c.env.o;
  PieceOut out;
  out.vol = (double)vol;
  out.mx = (double)mx * 0.25 + out.vol * o.x;
  out.my = (double)my * 0.25 + out.vol * o.y;
  out.mz = (double)mz * 0.25 + out.vol * o.z;
  out.chi = e.sv - e.se + sf - L;
  a.pout[p_slot] = out;
  PieceRef ref;
  ref.rec = base;
  ref.word = piece_word(e.nface, e.nedge, e.nrpv, cell_glue);
  a.pref[p_slot] = ref;
}

// Room for n records in the pool, from the calling lane: the first, or -1 when the pool is full.
__device__ inline int pool_records(const ShapeArgs& a, int n) {
  if (n == 0) return 0;
  const unsigned long long q = atomicAdd(&a.counters[C_REC_POOL], (unsigned long long)n);
  if (q + n > (unsigned long long)a.pool_cap) {
    atomicOr(a.status, ST_TABLE_FULL);
    return -1;
  }
  return (a.pcap / CHUNK) * REC_CHUNK + (int)q;
}

// A piece clipped outside its chunk's pass: terms to its slot, records to the pool.
template <typename CL>
__device__ __forceinline__ void emit_alone(CL& c, const ShapeDesc& sd, int tl, int p_slot, const ShapeArgs& a) {
  EmitAcc<CL> e;
  emit_scan(c, sd.nu + 14 * (size_t)tl, sd.L, e);
  const int base = pool_records(a, e.records());
  if (base >= 0) emit_out(c, sd, tl, e, p_slot, base, a);
}

// Hands piece slot p (or, with p = -1, every candidate of the tet) to the large-capacity kernel. first: the tet's
// first piece slot, or -1 when its candidates are still to be found.
__device__ inline void defer_item(const ShapeArgs& a, int shape, int t, int p, int first) {
  const unsigned long long idx = atomicAdd(&a.counters[C_DEFER_ITEMS], 1ull);
  if (idx < (unsigned long long)a.deferred_cap) a.deferred[idx] = make_int4(shape, t, p, first);
  else atomicOr(a.status, ST_TABLE_FULL);
}

// The next chunk of a split item: the next tet while tets are taken one at a time (up to single_end), else the next
// SUB tets. False past the item's last tet.
__device__ inline bool next_chunk(int& sub, int& sub_n, int& single_end, int ntb_all) {
  if (single_end > sub + 1) {
    sub += 1;
    sub_n = 1;
    return true;
  }
  if (single_end > sub) {  // the last single tet of its chunk: on with the chunk after it
    sub = single_end;
    single_end = 0;
  } else {
    sub += SUB;
  }
  if (sub >= ntb_all) return false;
  sub_n = min(SUB, ntb_all - sub);
  return true;
}

// ---------------------------------------------------------------------------------------------------------------
// clipping of one (tet, candidate) piece against the other candidates in order; returns CLIP_* for the piece
// ---------------------------------------------------------------------------------------------------------------
template <typename CL>
__device__ __forceinline__ int clip_piece(CL& cl, int m) {
  typedef typename CL::Real T;
  const TetEnv& env = cl.env;
  const float4 o = env.o;
  const double y1x = (double)env.tv[1].x - o.x, y1y = (double)env.tv[1].y - o.y, y1z = (double)env.tv[1].z - o.z;
  const double y2x = (double)env.tv[2].x - o.x, y2y = (double)env.tv[2].y - o.y, y2z = (double)env.tv[2].z - o.z;
  const double y3x = (double)env.tv[3].x - o.x, y3y = (double)env.tv[3].y - o.y, y3z = (double)env.tv[3].z - o.z;
  // CUT: the bisector against candidate c cuts the tet; SKIP: the tet lies in its kept half-space; else it lies outside
  enum { SKIP, CUT, OUTSIDE };
  auto classify = [&](int c, Plane<double>& P) {
    const float4 sj = env.cand_site(c);
    P = bisector64(env.si, sj, o);
    if (P.nx == 0.0 && P.ny == 0.0 && P.nz == 0.0) {  // concentric spheres: the larger one owns everything
      if (P.d > 0) return SKIP;
      // equal spheres: under the weight perturbation eps_i - eps_j the lower site id owns everything
      return P.d == 0 && env.site_i < env.cand_id(c) ? SKIP : OUTSIDE;
    }
    // the bisector's values at the tet vertices are exact in FP64
    const double h0 = P.d;
    const double h1 = fma(P.nx, y1x, fma(P.ny, y1y, fma(P.nz, y1z, P.d)));
    const double h2 = fma(P.nx, y2x, fma(P.ny, y2y, fma(P.nz, y2z, P.d)));
    const double h3 = fma(P.nx, y3x, fma(P.ny, y3y, fma(P.nz, y3z, P.d)));
    if (h0 > 0 && h1 > 0 && h2 > 0 && h3 > 0) return SKIP;
    if (h0 < 0 && h1 < 0 && h2 < 0 && h3 < 0) return OUTSIDE;
    return CUT;
  };
  cl.init_tet();
  Plane<double> P;
  if (CL::FEW_PLANES) {  // at most 28 candidates: find the cutting ones first, then every lane clips by its next one
    unsigned cut = 0;
    for (int c = 0; c < m; ++c) {
      if (c == env.ci) continue;
      const int k = classify(c, P);
      if (k == OUTSIDE) return CLIP_EMPTY;
      if (k == CUT) cut |= 1u << c;
    }
    for (; cut; cut &= cut - 1) {
      const int c = ctz_mask(cut);
      const int r = cl.clip(4 + c, round_plane<T>(bisector64(env.si, env.cand_site(c), o)));
      if (r != CLIP_OK) return r;
    }
    return CLIP_OK;
  }
  for (int c = 0; c < m; ++c) {
    if (c == env.ci) continue;
    const int k = classify(c, P);
    if (k == OUTSIDE) return CLIP_EMPTY;
    if (k == SKIP) continue;
    const int r = cl.clip(4 + c, round_plane<T>(P));
    if (r != CLIP_OK) return r;
  }
  return CLIP_OK;
}

// ---------------------------------------------------------------------------------------------------------------
// candidate kernel
// ---------------------------------------------------------------------------------------------------------------
__device__ inline double wave_min(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
  return v;
}
__device__ inline float wave_minf(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off));
  return v;
}
__device__ inline float wave_maxf(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// g_j at the four tet vertices (tet-local frame, exact in FP64)
__device__ __forceinline__ void g4(const float4* tv, const float4& s, double* g) {
  const float4 o = tv[0];
  double ax = (double)s.x - o.x, ay = (double)s.y - o.y, az = (double)s.z - o.z;
  double D = ax * ax + ay * ay + az * az - (double)s.w * s.w;
  g[0] = D;
  for (int v = 1; v < 4; ++v)
    g[v] = D - 2.0 * (((double)tv[v].x - o.x) * ax + ((double)tv[v].y - o.y) * ay + ((double)tv[v].z - o.z) * az);
}

// Drops the candidates that another candidate beats at all four tet vertices (g is affine, so then everywhere on the
// tet: the site owns nothing there and its bisector constrains no piece; the values are exact in FP64). The list is
// sorted by the power distance at the centroid, and a dominator has the smaller one, so rounds of three dominators
// taken in list order (each tested against the candidates after them) find the dominated candidates the three-at-a-time
// way; the rounds run while candidates remain past the dominators. Returns the new count; order is kept.
__device__ __forceinline__ int refine_candidates(const float4* tv, const float4* sites, unsigned char* cand, float* key,
                                                 int m) {
  for (int d = 0; d + 3 < m; d += 3) {
    double g0[4], g1[4], g2[4];
    g4(tv, sites[cand[d]], g0);
    g4(tv, sites[cand[d + 1]], g1);
    g4(tv, sites[cand[d + 2]], g2);
    int w = d + 3;
    for (int c = d + 3; c < m; ++c) {
      double g[4];
      g4(tv, sites[cand[c]], g);
      const bool dom = (g[0] > g0[0] && g[1] > g0[1] && g[2] > g0[2] && g[3] > g0[3]) ||
                       (g[0] > g1[0] && g[1] > g1[1] && g[2] > g1[2] && g[3] > g1[3]) ||
                       (g[0] > g2[0] && g[1] > g2[1] && g[2] > g2[2] && g[3] > g2[3]);
      if (!dom) {
        cand[w] = cand[c];
        key[w] = key[c];
        ++w;
      }
    }
    m = w;
  }
  return m;
}

// One wavefront per work item (a block, or a part of one). Latency-bound (site scans through the caches, FP64 values on
// a few dozen sites per tet); 17.5 KB of LDS, so nine items fit a compute unit.
__global__ __launch_bounds__(64) void k_candidates(ShapeArgs a) {
  static_assert(SLMAX <= 256, "candidate bytes index the site list");
  static_assert(TB * KRAW < 32768, "piece offsets are 16-bit");
  __shared__ float4 s_site[SLMAX];
  __shared__ int s_sid[SLMAX];
  __shared__ unsigned char s_cand[TB][KRAW];
  __shared__ float s_key[TB][KRAW];  // the candidates' sort keys
  __shared__ int s_m[TB];            // candidates of each tet; -1: left to the large-capacity kernel without a list
  __shared__ short s_off[TB + 1];
  __shared__ short s_order[TB];
  __shared__ int s_nsl;

  const int tid = threadIdx.x, lane = tid;
  const int nitems = a.nitems_dev ? *a.nitems_dev : a.nitems;
  unsigned long long n_cand = 0;
  // Work items are (shape, block or part of a block), ordered heaviest first. In a build the grid covers them, one
  // item per workgroup, and the hardware dispatcher hands them to compute units in that order as they free up,
  // which is the work queue. The passes of an incremental round read the item count on the device and launch a
  // grid sized to the resident workgroups, each taking items in grid-stride order.
  for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
  const unsigned long long clock0 = wall_clock64();
  const int2 wi = a.items[item];
  const int shape = __builtin_amdgcn_readfirstlane(wi.x & 0xffff);
  const ShapeDesc sd = a.shapes[shape];
  const int blk = wi.y & ((1 << ITEM_PART_SHIFT) - 1), part = wi.y >> ITEM_PART_SHIFT;
  // the tets of the item to clip, relative to its first tet (an incremental update names the tets a new sphere can
  // reach; every other item takes all)
  const unsigned tet_mask16 = (unsigned)wi.x >> 16;
  const unsigned long long item_mask = tet_mask16 ? (unsigned long long)tet_mask16 : ~0ull;
  int tb0 = sd.blk[blk];
  int ntb_all = sd.blk[blk + 1] - tb0;
  if (part > 0) {  // one part of a heavy block (the host only makes parts that exist)
    tb0 += (part - 1) * SPLIT_TETS;
    ntb_all = min(SPLIT_TETS, ntb_all - (part - 1) * SPLIT_TETS);
  }
  // A block whose shared site list overflows is redone in chunks of SUB tets (smaller boxes, shorter lists), and a
  // chunk that still overflows one tet at a time, each with its own candidates found among all of the shape's
  // sites. A tet then goes to the large-capacity kernel only for reasons that depend on its own candidates (more
  // than fit the list, or the clip budget), never on its neighbours' or on sites that own nothing in it: an
  // incremental update, which recomputes a tet's pieces to take them back, must take the path that added them.
  int sub = 0, sub_n = ntb_all, single_end = 0;  // tets [sub, single_end): one at a time
  bool split = false;
  while (true) {
  const int t0 = tb0 + sub;
  const int ntb = sub_n;
  const bool single = single_end > sub;
  const unsigned long long cmask = item_mask >> sub;  // bit lt: tet t0 + lt is clipped
  if (split && !(cmask & (ntb >= 64 ? ~0ull : (1ull << ntb) - 1ull))) {  // a chunk without such tets
    if (!next_chunk(sub, sub_n, single_end, ntb_all)) break;
    continue;
  }
  int tpt = 1;  // lanes per tet in the candidate phase
  while (tpt < 64 && 2 * tpt * ntb <= 64) tpt *= 2;

  // ---- 1. the tets' bounding box 
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  {
    if (!single && tid < ntb && ((cmask >> tid) & 1ull)) {
      const float4* tp = sd.tp + 4 * (size_t)(t0 + tid);
      for (int v = 0; v < 4; ++v) {
        float4 p = tp[v];
        lo[0] = fminf(lo[0], p.x);
        lo[1] = fminf(lo[1], p.y);
        lo[2] = fminf(lo[2], p.z);
        hi[0] = fmaxf(hi[0], p.x);
        hi[1] = fmaxf(hi[1], p.y);
        hi[2] = fmaxf(hi[2], p.z);
      }
    }
  }
  for (int k = 0; k < 3; ++k) {
    lo[k] = wave_minf(lo[k]);
    hi[k] = wave_maxf(hi[k]);
  }
  s_m[tid] = 0;
  if (tid == 0) s_nsl = 0;
  __syncthreads();

  // ---- 2. sites that can own a point of the box: min over the box of g_j <= min over j of max over the box
  //        (g_j(x) = d_j(x) - |x - o|^2 is affine; values exact in FP64); for a single tet, the same test on the
  //        tet itself (its exact candidates)
  const float4* ssite = a.site + sd.site_off;
  if (single) {
    const float4* tv = sd.tp + 4 * (size_t)t0;
    const float4 o = tv[0];
    double y[3][3];
    for (int v = 1; v < 4; ++v) {
      y[v - 1][0] = (double)tv[v].x - o.x;
      y[v - 1][1] = (double)tv[v].y - o.y;
      y[v - 1][2] = (double)tv[v].z - o.z;
    }
    // the five dominators of the candidate phase among all of the shape's sites (lowest index on ties): the site
    // attaining U and the owner of each vertex; a site one of them beats at all four vertices is not collected, so
    // that the list holds the tet's exact candidates less those (which the candidate phase drops anyway)
    double dv[5];
    int dj[5];
    for (int k = 0; k < 5; ++k) {
      dv[k] = INFINITY;
      dj[k] = 0x7fffffff;
    }
    for (int j = tid; j < sd.ns; j += 64) {
      const float4 s = ssite[j];
      const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
      double gq[4];
      gq[0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
      for (int v = 0; v < 3; ++v) gq[v + 1] = gq[0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
      const double gmx = fmax(fmax(gq[0], gq[1]), fmax(gq[2], gq[3]));
      for (int k = 0; k < 5; ++k) {
        const double x = k == 0 ? gmx : gq[k - 1];
        if (x < dv[k] || (x == dv[k] && j < dj[k])) {
          dv[k] = x;
          dj[k] = j;
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1)
      for (int k = 0; k < 5; ++k) {
        const double x2 = __shfl_xor(dv[k], off);
        const int j2 = __shfl_xor(dj[k], off);
        if (x2 < dv[k] || (x2 == dv[k] && j2 < dj[k])) {
          dv[k] = x2;
          dj[k] = j2;
        }
      }
    const double U = dv[0];
    double gb[5][4];
    for (int k = 0; k < 5; ++k) {
      const float4 s = ssite[dj[k]];
      const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
      gb[k][0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
      for (int v = 0; v < 3; ++v) gb[k][v + 1] = gb[k][0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
    }
    for (int j = tid; j < sd.ns; j += 64) {
      const float4 s = ssite[j];
      const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
      double g[4];
      g[0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
      for (int v = 0; v < 3; ++v) g[v + 1] = g[0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
      const double gmn = fmin(fmin(g[0], g[1]), fmin(g[2], g[3]));
      bool dom = false;
      for (int k = 0; k < 5; ++k)
        dom = dom || (g[0] > gb[k][0] && g[1] > gb[k][1] && g[2] > gb[k][2] && g[3] > gb[k][3]);
      if (gmn <= U && !dom) {
        const int q = atomicAdd(&s_nsl, 1);
        if (q < SLMAX) {
          s_site[q] = s;
          s_sid[q] = sd.site_off + j;
        }
      }
    }
  } else {
  const double bx = lo[0], by = lo[1], bz = lo[2];
  const double ex = (double)hi[0] - bx, ey = (double)hi[1] - by, ez = (double)hi[2] - bz;
  double umin = INFINITY;
  for (int j = tid; j < sd.ns; j += 64) {
    float4 s = ssite[j];
    double ax_ = (double)s.x - bx, ay_ = (double)s.y - by, az_ = (double)s.z - bz;
    double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
    double gmax = D + fmax(0.0, -2.0 * ex * ax_) + fmax(0.0, -2.0 * ey * ay_) + fmax(0.0, -2.0 * ez * az_);
    umin = fmin(umin, gmax);
  }
  const double UB = wave_min(umin);
  for (int j = tid; j < sd.ns; j += 64) {
    float4 s = ssite[j];
    double ax_ = (double)s.x - bx, ay_ = (double)s.y - by, az_ = (double)s.z - bz;
    double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
    double gmin = D + fmin(0.0, -2.0 * ex * ax_) + fmin(0.0, -2.0 * ey * ay_) + fmin(0.0, -2.0 * ez * az_);
    if (gmin <= UB) {
      int q = atomicAdd(&s_nsl, 1);
      if (q < SLMAX) {
        s_site[q] = s;
        s_sid[q] = sd.site_off + j;
      }
    }
  }
  }
  __syncthreads();
  const int nsl = s_nsl;
  if (nsl > SLMAX && !(a.flags & RPD_FORCE_SLOW_PATH)) {
    if (!split && ntb > SUB) {  // chunks of SUB tets
      split = true;
      sub_n = SUB;
      if (tid == 0) stat_add(a, C_SPLIT, 1ull);
      __syncthreads();
      continue;
    }
    if (!single) {  // one tet at a time, each with its exact candidates
      split = true;
      single_end = sub + ntb;
      sub_n = 1;
      __syncthreads();
      continue;
    }
  }
  const bool block_overflow = nsl > SLMAX || (a.flags & RPD_FORCE_SLOW_PATH);

  // ---- 3. candidates of every tet: sites whose minimum over the tet is <= min_j max over the tet
  if (!block_overflow) {
    const int lt = tid / tpt, h = tid % tpt;
    if (lt < ntb && ((cmask >> lt) & 1ull)) {
      const float4* tv = sd.tp + 4 * (size_t)(t0 + lt);
      const float4 o = tv[0];
      double y[3][3];
      for (int v = 1; v < 4; ++v) {
        y[v - 1][0] = (double)tv[v].x - o.x;
        y[v - 1][1] = (double)tv[v].y - o.y;
        y[v - 1][2] = (double)tv[v].z - o.z;
      }
      const double ycx = (y[0][0] + y[1][0] + y[2][0]) * 0.25, ycy = (y[0][1] + y[1][1] + y[2][1]) * 0.25,
                   ycz = (y[0][2] + y[1][2] + y[2][2]) * 0.25;
      // five dominators, each a site with its list position and id (the lowest id on ties, so that the choice does
      // not depend on the list's order): [0] attains U = min over sites of the maximum of g over the tet, [1 + v]
      // the minimum of g at vertex v (that vertex's owner)
      double dv[5];
      int dq[5], did[5];
      for (int k = 0; k < 5; ++k) {
        dv[k] = INFINITY;
        dq[k] = 0;
        did[k] = 0x7fffffff;
      }
      for (int q = h; q < nsl; q += tpt) {
        float4 s = s_site[q];
        double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        double gq[4];
        gq[0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        for (int v = 0; v < 3; ++v) gq[v + 1] = gq[0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
        const double gmx = fmax(fmax(gq[0], gq[1]), fmax(gq[2], gq[3]));
        const int id = s_sid[q];
        for (int k = 0; k < 5; ++k) {
          const double x = k == 0 ? gmx : gq[k - 1];
          if (x < dv[k] || (x == dv[k] && id < did[k])) {
            dv[k] = x;
            dq[k] = q;
            did[k] = id;
          }
        }
      }
      for (int off = 1; off < tpt; off <<= 1)
        for (int k = 0; k < 5; ++k) {
          const double x2 = __shfl_xor(dv[k], off);
          const int q2 = __shfl_xor(dq[k], off), id2 = __shfl_xor(did[k], off);
          if (x2 < dv[k] || (x2 == dv[k] && id2 < did[k])) {
            dv[k] = x2;
            dq[k] = q2;
            did[k] = id2;
          }
        }
      const double U = dv[0];
      if (a.tet_U && sd.sign > 0 && h == 0) a.tet_U[sd.tet_off + t0 + lt] = U;
      // the dominators' g at the four vertices: a site that one of them beats at all four owns no point of the tet
      // and its bisector constrains no piece (the dominator is a candidate, and its own bisector already does), so
      // it is not a candidate; the same test among all candidates follows once they are sorted
      double gb[5][4];
      for (int k = 0; k < 5; ++k) {
        const float4 s = s_site[dq[k]];
        const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        gb[k][0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        for (int v = 0; v < 3; ++v) gb[k][v + 1] = gb[k][0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
      }
      for (int q = h; q < nsl; q += tpt) {
        float4 s = s_site[q];
        double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        double g[4];
        g[0] = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        for (int v = 0; v < 3; ++v) g[v + 1] = g[0] - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
        const double gmn = fmin(fmin(g[0], g[1]), fmin(g[2], g[3]));
        bool dom = false;
        for (int k = 0; k < 5; ++k)
          dom = dom || (g[0] > gb[k][0] && g[1] > gb[k][1] && g[2] > gb[k][2] && g[3] > gb[k][3]);
        const double D = g[0];
        if (gmn <= U && !dom) {
          int pos = atomicAdd(&s_m[lt], 1);
          if (pos < KRAW) {
            s_cand[lt][pos] = (unsigned char)q;
            s_key[lt][pos] = (float)(D - 2.0 * (ycx * ax_ + ycy * ay_ + ycz * az_));
          }
        }
      }
    }
  }
  __syncthreads();
  // sort each tet's candidates by (power distance at the centroid, site id) and drop the dominated ones
  if (tid < ntb && ((cmask >> tid) & 1ull)) {
    int m = s_m[tid];
    if (!block_overflow && m <= KRAW) {
      for (int x = 1; x < m; ++x) {
        const float kx = s_key[tid][x];
        const unsigned char cx = s_cand[tid][x];
        const int ix = s_sid[cx];
        int y = x - 1;
        while (y >= 0 && (s_key[tid][y] > kx || (s_key[tid][y] == kx && s_sid[s_cand[tid][y]] > ix))) {
          s_key[tid][y + 1] = s_key[tid][y];
          s_cand[tid][y + 1] = s_cand[tid][y];
          --y;
        }
        s_key[tid][y + 1] = kx;
        s_cand[tid][y + 1] = cx;
      }
      m = refine_candidates(sd.tp + 4 * (size_t)(t0 + tid), s_site, s_cand[tid], s_key[tid], m);
    }
    // a tet over the budget goes to the large-capacity kernel, with its sorted, refined candidates when they fit the
    // list (else that kernel finds them among all sites); either way the choice depends on its own candidates only
    if (block_overflow || m > a.kmax) stat_add(a, block_overflow ? C_DEFER_BLOCK : C_DEFER_KMAX, 1ull);
    if (block_overflow || m > KRAW) {
      m = -1;
      defer_item(a, shape, t0 + tid, -1, -1);
    }
    s_m[tid] = m;
  }
  __syncthreads();
  // pieces are laid out tet by tet with the tets ordered by candidate count, largest first: every piece of a tet
  // loops over the same planes, so a wavefront's lanes then have similar trip counts
  {
    const int mt = tid < ntb ? max(s_m[tid], 0) : 0;
    int rank = 0, off = 0;
    for (int u = 0; u < TB; ++u) {
      const int mu = __shfl(mt, u);
      if (mu > mt || (mu == mt && u < tid)) {
        ++rank;
        off += mu;
      }
    }
    s_order[rank] = (short)tid;
    s_off[rank] = (short)off;
    if (rank == TB - 1) s_off[TB] = (short)(off + mt);
  }
  __syncthreads();
  const int npairs = s_off[TB];
  int base = 0;
  if (lane == 0 && npairs) {
    const unsigned long long q = atomicAdd(&a.counters[C_PIECE_SLOTS], (unsigned long long)npairs);
    base = q + npairs <= (unsigned long long)a.pcap ? (int)q : -1;
    if (base < 0) atomicOr(a.status, ST_TABLE_FULL);
  }
  base = __builtin_amdgcn_readfirstlane(base);
  if (base >= 0) {
    for (int p = tid; p < npairs; p += 64) {
      int lo_ = 0, hi_ = TB - 1;  // last position j with s_off[j] <= p
      while (lo_ < hi_) {
        const int mid = (lo_ + hi_ + 1) >> 1;
        if (s_off[mid] <= p) lo_ = mid;
        else hi_ = mid - 1;
      }
      const int lt = s_order[lo_], first = s_off[lo_], m = s_m[lt];
      a.psite[base + p] = s_sid[s_cand[lt][p - first]];
      PieceDesc d;
      d.t = t0 + lt;
      d.shape = shape;
      d.first = base + first;
      d.m = m;
      a.pdesc[base + p] = d;
      if (p == first && a.tet_slots) a.tet_slots[sd.tet_off + t0 + lt] = make_int2(base + first, m);
      if (m > a.kmax) {
        if (p == first) defer_item(a, shape, t0 + lt, -1, base + first);
      } else {
        ++n_cand;
      }
    }
  }
  if (!split || !next_chunk(sub, sub_n, single_end, ntb_all)) break;
  __syncthreads();  // the next chunk reuses every shared array
  }
  __syncthreads();  // the next item reuses every shared array
  if (a.item_cost && tid == 0)  // the item's duration (every thread is past it), a scheduling hint for the next build
    a.item_cost[item] = (unsigned)min(wall_clock64() - clock0, 0xffffffffull);
  }
  for (int off = 32; off > 0; off >>= 1) n_cand += __shfl_xor(n_cand, off);
  if (lane == 0 && n_cand) stat_add(a, C_CAND, n_cand);
}

// ---------------------------------------------------------------------------------------------------------------
// piece kernel
// ---------------------------------------------------------------------------------------------------------------
// Vertex slots per piece: 16 (19.7 KB of LDS a wavefront in FP32) or 12 (15.6 KB: more wavefronts fit a compute unit).
// A piece that outgrows them is redone after its chunk with a 64-slot polytope; the arithmetic is the same.
//
// A piece's terms are plain stores, no value of which the kernel waits for: with the sums and the element pieces
// entered into hash tables here, a chunk spent most of its time on the round trips of those dependent atomics.
constexpr int WIN = CHUNK + 2 * KRAW;  // candidate slots of the tets that a chunk touches

template <typename T, int SLOTS>
__global__ __launch_bounds__(64) void k_clip_pieces(ShapeArgs a) {
  typedef typename StoreOf<T, Topo32, SLOTS>::type PolyStore;
  __shared__ __attribute__((aligned(16))) unsigned char s_poly[PolyStore::coord_bytes(64)];
  __shared__ unsigned s_topo[SLOTS * 64];
  __shared__ float4 s_csite[WIN];
  __shared__ int s_csid[WIN];
  __shared__ int s_over[CHUNK];  // this chunk's pieces that ran out of vertex slots
  __shared__ int s_nover;
  if (*a.status & ST_TABLE_FULL) return;  // some slots were never filled; the call is redone with larger buffers
  const int lane = threadIdx.x;
  const int np_all = (int)min(a.counters[C_PIECE_SLOTS], (unsigned long long)a.pcap);
  const int nchunks = (np_all + CHUNK - 1) / CHUNK;
  if (lane == 0) {
    s_nover = 0;
    if (blockIdx.x == 0) a.counters[C_CHUNKS] = (unsigned long long)nchunks;
  }
  long long n_pairs = 0;
  unsigned long long n64 = 0;
  for (int chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x) {
    const int p = chunk * CHUNK + lane;
    const int last = min(CHUNK, np_all - chunk * CHUNK) - 1;
    PieceDesc d = a.pdesc[chunk * CHUNK + min(lane, last)];
    const bool run = lane <= last && d.m <= a.kmax;
    // the candidates of the chunk's tets are consecutive slots
    const int w0 = __shfl(d.first, 0), w1 = min(__shfl(d.first + d.m, last), w0 + WIN);
    __syncthreads();
    for (int q = w0 + lane; q < w1; q += 64) {
      const int s = a.psite[q];
      s_csid[q - w0] = s;
      s_csite[q - w0] = a.site[s];
    }
    __syncthreads();
    const ShapeDesc& sd = a.shapes[d.shape];
    const int co = d.first - w0;
    auto bind = [&](TetEnv& env, int t, int c0, int ci) {
      env.tv = sd.tp + 4 * (size_t)t;
      env.o = env.tv[0];
      env.face64 = sd.tf + 4 * (size_t)t;
      env.sid = s_csid + c0;
      env.csite = s_csite + c0;
      env.site = nullptr;
      env.ncs = INT_MAX;
      env.ci = ci;
      env.si = env.csite[ci];
      env.site_i = env.sid[ci];
    };
    typedef Clipper<T, Topo32, unsigned, SLOTS, false, RegTab> CL;
    CL cl;
    EmitAcc<CL> e;
    e.nface = e.nedge = e.nrpv = 0;
    int r = CLIP_EMPTY;
    if (run) {
      cl.st.bind(s_poly, s_topo, lane, 64);
      cl.tab.clear(0);
      cl.a = nullptr;  // only the exact predicates use it (not compiled into this kernel)
      cl.flags = a.flags;
      cl.np = 4 + d.m;
      cl.n64 = 0;
      cl.nex = 0;
      bind(cl.env, d.t, co, p - d.first);
      r = clip_piece(cl, d.m);
      n64 += cl.n64;
      if (r == CLIP_OK) {
        n_pairs += sd.sign;  // live pieces
        emit_scan(cl, sd.nu + 14 * (size_t)d.t, sd.L, e);
      } else {
        a.pref[p].word = 0;
        if (r == CLIP_DEFER) {
          stat_add(a, C_DEFER_CLIP, 1ull);
          defer_item(a, d.shape, d.t, p, d.first);
        } else if (r == CLIP_FULL) {
          s_over[atomicAdd(&s_nover, 1)] = lane;
        }
      }
    }
    // records: the lanes' runs one after the other, in the chunk's own range when they fit
    const int n = e.records();
    int incl = n;
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    const int total = __shfl(incl, 63);
    int base = chunk * REC_CHUNK;
    if (total > REC_CHUNK) {
      int q = 0;
      if (lane == 0) q = pool_records(a, total);
      base = __builtin_amdgcn_readfirstlane(q);
    }
    if (lane == 0) a.chunk_recs[chunk] = total > REC_CHUNK ? 0 : total;
    if (run && r == CLIP_OK && base >= 0) emit_out(cl, sd, d.t, e, p, base + incl - n, a);
    // Pieces that ran out of vertex slots are redone here, one per lane, with a BIG_VCAP-slot polytope. The chunk's
    // small polytopes are dead by now, so the first records live in their LDS; more go to a global-memory pool (same
    // arithmetic, same bits). Which path computes a piece must depend on the piece alone (an incremental update must
    // take back exactly the bits it added), so a full pool is a table overflow (the call is redone with larger
    // buffers), never a deferral.
    __syncthreads();
    const int nover = s_nover;
    if (nover) {
      if (lane < nover) {
        const int src = s_over[lane];
        const int pb = chunk * CHUNK + src;
        const PieceDesc db = a.pdesc[pb];
        const ShapeDesc& sb = a.shapes[db.shape];
        const int m = db.m;
        constexpr size_t CB = sizeof(typename Coord4<T>::type) * BIG_VCAP;
        constexpr size_t REC = (CB + 8 * BIG_VCAP + 64 + 15) / 16 * 16;
        constexpr int NLDS = (int)(sizeof(s_poly) / REC);
        static_assert(CB + 8 * BIG_VCAP + 32 <= BIG_BYTES, "large-capacity polytope record");
        const unsigned long long slot = atomicAdd(&a.counters[C_BIG], 1ull);
        if (lane >= NLDS && slot >= (unsigned long long)a.big_cap) {
          atomicOr(a.status, ST_TABLE_FULL);
        } else {
          unsigned char* b = lane < NLDS ? s_poly + (size_t)lane * REC : a.big + slot * BIG_BYTES;
          Clipper<T, Topo64, unsigned long long, BIG_VCAP, false, MemTab> cb;
          cb.st.c = reinterpret_cast<typename Coord4<T>::type*>(b);
          cb.st.w = reinterpret_cast<unsigned long long*>(b + CB);
          cb.st.stride = 1;
          cb.tab.base = b + CB + 8 * BIG_VCAP;
          cb.tab.stride = 1;
          cb.tab.clear(4 + m);
          cb.a = nullptr;
          cb.flags = a.flags;
          cb.np = 4 + m;
          cb.n64 = 0;
          cb.nex = 0;
          {
            cb.env.tv = sb.tp + 4 * (size_t)db.t;
            cb.env.o = cb.env.tv[0];
            cb.env.face64 = sb.tf + 4 * (size_t)db.t;
            cb.env.sid = s_csid + (db.first - w0);
            cb.env.csite = s_csite + (db.first - w0);
            cb.env.site = nullptr;
            cb.env.ncs = INT_MAX;
            cb.env.ci = pb - db.first;
            cb.env.si = cb.env.csite[cb.env.ci];
            cb.env.site_i = cb.env.sid[cb.env.ci];
          }
          const int rb = clip_piece(cb, m);
          n64 += cb.n64;
          if (rb == CLIP_OK) {
            n_pairs += sb.sign;
            emit_alone(cb, sb, db.t, pb, a);
          } else if (rb != CLIP_EMPTY) {  // a predicate undecided in FP64, or over BIG_VCAP vertices
            stat_add(a, C_DEFER_CLIP, 1ull);
            defer_item(a, db.shape, db.t, pb, db.first);
          }
        }
      }
      __syncthreads();
      if (lane == 0) s_nover = 0;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    n_pairs += __shfl_xor(n_pairs, off);
    n64 += __shfl_xor(n64, off);
  }
  if (lane == 0) {
    if (n_pairs) stat_add(a, C_PAIRS, (unsigned long long)n_pairs);  // in two's complement
    if (n64) stat_add(a, C_FP64, n64);
  }
}

// ---------------------------------------------------------------------------------------------------------------
// large-capacity kernel: one wavefront per deferred item, FP64 constructions, exact predicates, global scratch
// ---------------------------------------------------------------------------------------------------------------
struct SlowScratch {  // per wave, in global memory: the candidate lists, their vertex values, the global-memory polytopes
  static constexpr size_t cand_bytes = SLOW_KMAX * sizeof(int);
  static constexpr size_t key_bytes = SLOW_KMAX * sizeof(double);
  static constexpr size_t g_bytes = SLOW_KMAX * 4 * sizeof(double);   // g_j at the four tet vertices
  static constexpr size_t wave_bytes = 2 * (cand_bytes + key_bytes) + g_bytes;  // unsorted and sorted lists
  static constexpr size_t xyz_bytes = 64 * SLOW_VMAX * sizeof(Coord4<double>::type);  // [slot][lane]
  static constexpr size_t topo_bytes = 64 * SLOW_VMAX * sizeof(unsigned long long);    // [slot][lane]
  static constexpr size_t tab_bytes = 64 * (size_t)SLOW_PMAX;                          // [plane][lane]
  static constexpr size_t bytes = wave_bytes + xyz_bytes + topo_bytes + tab_bytes;
};
constexpr int SLOW_LDS_ITEMS = 512;  // the first deferred items go to the LDS variant (one item per wave)

// The LDS variant (few items: latency) keeps the candidate lists and 32 lanes' polytopes (32 vertices) in LDS; an item
// with more than 256 candidates, or a piece with more vertices, is handed to the global variant through the overflow
// list. The global variant (many items: throughput) keeps the lists and all 64 lanes' polytopes (64 vertices) in its
// scratch and takes the items past the LDS variant's share, then the overflow list.
template <bool LDS>
struct SlowCfg;
template <>
struct SlowCfg<true> {
  static constexpr int CL = 32, VCAP = 32, KCAP = 256;
  typedef unsigned Mask;
};
template <>
struct SlowCfg<false> {
  static constexpr int CL = 64, VCAP = SLOW_VMAX, KCAP = SLOW_KMAX;
  typedef unsigned long long Mask;
};

__device__ inline void push_overflow(const ShapeArgs& a, int4 item) {
  const unsigned long long idx = atomicAdd(&a.counters[C_DEFER2], 1ull);
  if (idx < (unsigned long long)a.deferred2_cap) a.deferred2[idx] = item;
  else atomicOr(a.status, ST_TABLE_FULL);
}

// One wavefront per deferred item: the lanes split the scan over all of the shape's sites (candidates are
// compacted in ascending site order by ballots), drop dominated candidates and rank-sort the rest, then clip the
// pieces with FP64 polytopes (lanes interleaved slot by slot).
template <bool LDS>
__global__ __launch_bounds__(64, LDS ? 1 : 2) void k_clip_slow(ShapeArgs a, unsigned char* scratch, int item_begin, int item_end) {
  typedef SlowCfg<LDS> C;
  constexpr int CL = C::CL, KC = C::KCAP;
  __shared__ Coord4<double>::type s_xyz[LDS ? C::VCAP * CL : 1];
  __shared__ unsigned long long s_topo[LDS ? C::VCAP * CL : 1];
  __shared__ unsigned char s_tab[LDS ? (4 + KC) * CL : 1];
  __shared__ int s_cand[LDS ? 2 * KC : 1];
  __shared__ double s_key[LDS ? 6 * KC : 1];
  // on-chip copies for the clipping loop, whose plane rebuilds would otherwise wait on memory: the item's tet and
  // the sites of its first SC candidates (sorted positions)
  constexpr int SC = 256;
  __shared__ float4 s_tv4[4];
  __shared__ double4 s_tf4[4];
  __shared__ float4 s_csite[SC];
  if (*a.status & ST_TABLE_FULL) return;  // the call is redone with larger buffers
  const int n_main = (int)min(min(a.counters[C_DEFER_ITEMS], (unsigned long long)a.deferred_cap),
                              (unsigned long long)item_end);
  const int n_over = LDS ? 0 : (int)min(a.counters[C_DEFER2], (unsigned long long)a.deferred2_cap);
  const int n_items = max(n_main - item_begin, 0) + n_over;
  const int lane = threadIdx.x;
  unsigned char* wbase = scratch + (size_t)blockIdx.x * SlowScratch::bytes;
  int* cand = LDS ? s_cand : (int*)wbase;
  int* scand = LDS ? s_cand + KC : (int*)(wbase + SlowScratch::cand_bytes + SlowScratch::key_bytes);
  double* key = LDS ? s_key : (double*)(wbase + SlowScratch::cand_bytes);
  double* skey = LDS ? s_key + KC : (double*)(wbase + 2 * SlowScratch::cand_bytes + SlowScratch::key_bytes);
  double* gv = LDS ? s_key + 2 * KC : (double*)(wbase + 2 * (SlowScratch::cand_bytes + SlowScratch::key_bytes));
  const int cl_lane = lane < CL ? lane : 0;
  Coord4<double>::type* xyz =
      LDS ? s_xyz + cl_lane : (Coord4<double>::type*)(wbase + SlowScratch::wave_bytes) + cl_lane;
  unsigned long long* topo =
      LDS ? s_topo + cl_lane
          : (unsigned long long*)(wbase + SlowScratch::wave_bytes + SlowScratch::xyz_bytes) + cl_lane;
  unsigned char* tab =
      LDS ? s_tab + cl_lane : wbase + SlowScratch::wave_bytes + SlowScratch::xyz_bytes + SlowScratch::topo_bytes + cl_lane;
  unsigned long long n_pairs = 0, n64 = 0, nex = 0;
  for (int vi = blockIdx.x; vi < n_items; vi += gridDim.x) {
    const int main_count = max(n_main - item_begin, 0);
    const int4 di = vi < main_count ? a.deferred[item_begin + vi] : a.deferred2[vi - main_count];
    const ShapeDesc sd = a.shapes[__builtin_amdgcn_readfirstlane(di.x)];
    const int t = di.y;
    const int want = di.z;  // piece slot, or -1: every candidate of the tet
    int first = di.w;       // the tet's first piece slot, or -1: its candidates are found here
    const float4* ssite = a.site + sd.site_off;
    float4 tv[4];
    for (int v = 0; v < 4; ++v) tv[v] = sd.tp[4 * (size_t)t + v];
    if (lane < 4) {
      s_tv4[lane] = sd.tp[4 * (size_t)t + lane];
      s_tf4[lane] = sd.tf[4 * (size_t)t + lane];
    }
    const float4 o = tv[0];
    double y[3][3];
    for (int v = 1; v < 4; ++v) {
      y[v - 1][0] = (double)tv[v].x - o.x;
      y[v - 1][1] = (double)tv[v].y - o.y;
      y[v - 1][2] = (double)tv[v].z - o.z;
    }
    const double ycx = (y[0][0] + y[1][0] + y[2][0]) * 0.25, ycy = (y[0][1] + y[1][1] + y[2][1]) * 0.25,
                 ycz = (y[0][2] + y[1][2] + y[2][2]) * 0.25;
    // a tet's sorted candidates come with its piece slots when they fit the candidate kernel's list (a function of
    // the tet's candidates only); otherwise they are found here among all sites
    int m = 0;
    if (first >= 0) {
      m = a.pdesc[first].m;
      if (LDS && m > KC) {  // (a tet whose candidates this kernel's global variant found)
        if (lane == 0) push_overflow(a, di);
        continue;
      }
      for (int x = lane; x < m; x += 64) {
        const int sx = a.psite[first + x];
        scand[x] = sx;
        if (x < SC) s_csite[x] = a.site[sx];
      }
      __syncthreads();
    } else {
      // candidates among ALL sites of the shape (same exact test as the fast kernel)
      double U = INFINITY;
      for (int j = lane; j < sd.ns; j += 64) {
        float4 s = ssite[j];
        double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        double gmx = D;
        for (int v = 0; v < 3; ++v) gmx = fmax(gmx, D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_));
        U = fmin(U, gmx);
      }
      for (int off = 32; off > 0; off >>= 1) U = fmin(U, __shfl_xor(U, off));
      if (a.tet_U && sd.sign > 0 && lane == 0) a.tet_U[sd.tet_off + t] = U;
      for (int base = 0; base < sd.ns; base += 64) {
        const int j = base + lane;
        bool take = false;
        double kk = 0.0;
        if (j < sd.ns) {
          float4 s = ssite[j];
          double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
          double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
          double gmn = D;
          for (int v = 0; v < 3; ++v) gmn = fmin(gmn, D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_));
          take = gmn <= U;
          kk = D - 2.0 * (ycx * ax_ + ycy * ay_ + ycz * az_);
        }
        unsigned long long mask = __ballot(take);
        int pos = m + __popcll(mask & ((1ull << lane) - 1ull));
        if (take && pos < KC) {
          cand[pos] = sd.site_off + j;
          key[pos] = kk;
        }
        m += __popcll(mask);
      }
      if (m > KC) {
        if (lane == 0) {
          if (LDS) push_overflow(a, di);
          else atomicOr(a.status, ST_SLOW_CAPACITY);
        }
        continue;
      }
      __syncthreads();
      // drop every candidate that another one beats at all four tet vertices (g is affine, so then everywhere on the
      // tet: it owns nothing and its bisector constrains no piece); the values are exact in FP64
      for (int x = lane; x < m; x += 64) {
        const float4 s = a.site[cand[x]];
        const double ax_ = (double)s.x - o.x, ay_ = (double)s.y - o.y, az_ = (double)s.z - o.z;
        const double D = ax_ * ax_ + ay_ * ay_ + az_ * az_ - (double)s.w * s.w;
        gv[4 * x] = D;
        for (int v = 0; v < 3; ++v) gv[4 * x + 1 + v] = D - 2.0 * (y[v][0] * ax_ + y[v][1] * ay_ + y[v][2] * az_);
      }
      __syncthreads();
      int kept = 0;
      for (int base = 0; base < m; base += 64) {
        const int x = base + lane;
        bool keep = false;
        double kx = 0.0;
        int cx = 0;
        if (x < m) {
          const double g0 = gv[4 * x], g1 = gv[4 * x + 1], g2 = gv[4 * x + 2], g3 = gv[4 * x + 3];
          keep = true;
          for (int q = 0; q < m && keep; ++q)
            keep = !(gv[4 * q] < g0 && gv[4 * q + 1] < g1 && gv[4 * q + 2] < g2 && gv[4 * q + 3] < g3);
          kx = key[x];
          cx = cand[x];
        }
        const unsigned long long mask = __ballot(keep);
        __syncthreads();  // every lane has read cand/key of this chunk before they are overwritten in place
        if (keep) {
          const int pos = kept + __popcll(mask & ((1ull << lane) - 1ull));
          cand[pos] = cx;
          key[pos] = kx;
        }
        kept += __popcll(mask);
      }
      m = kept;
      __syncthreads();
      // rank sort by (key, position): positions ascend with the site id, so ties keep the site order
      for (int x = lane; x < m; x += 64) {
        const double kx = key[x];
        int rank = 0;
        for (int q = 0; q < m; ++q) {
          const double kq = key[q];
          rank += (kq < kx || (kq == kx && q < x)) ? 1 : 0;
        }
        scand[rank] = cand[x];
        skey[rank] = kx;
        if (rank < SC) s_csite[rank] = a.site[cand[x]];
      }
      // piece slots for the tet's candidates
      __syncthreads();
      int q = -1;
      if (lane == 0) {
        const unsigned long long at = atomicAdd(&a.counters[C_PIECE_SLOTS], (unsigned long long)m);
        if (at + m <= (unsigned long long)a.pcap) q = (int)at;
        else atomicOr(a.status, ST_TABLE_FULL);
      }
      first = __builtin_amdgcn_readfirstlane(q);
      if (first < 0) continue;
      if (lane == 0 && a.tet_slots) a.tet_slots[sd.tet_off + t] = make_int2(first, m);
      for (int x = lane; x < m; x += 64) {
        PieceDesc d;
        d.t = t;
        d.shape = di.x;
        d.first = first;
        d.m = m;
        a.pdesc[first + x] = d;
        a.psite[first + x] = scand[x];
        a.pref[first + x].word = 0;
      }
    }
    if (lane < CL)
      for (int k = 0; k < 4 + m; ++k) tab[CL * k] = 0;  // the plane ids of this item start unpaired
    __syncthreads();
    for (int ci = lane; ci < m && lane < CL; ci += CL) {
      if (want >= 0 && first + ci != want) continue;
      Clipper<double, Topo64, typename C::Mask, C::VCAP, true, MemTab> cl;
      cl.st.c = xyz;
      cl.st.w = topo;
      cl.st.stride = CL;
      cl.tab = MemTab{tab, CL};
      cl.a = &a;
      cl.flags = a.flags & ~RPD_FORCE_FP64;
      cl.np = 4 + m;
      cl.n64 = 0;
      cl.nex = 0;
      cl.env.tv = s_tv4;
      cl.env.o = s_tv4[0];
      cl.env.face64 = s_tf4;
      cl.env.sid = scand;
      cl.env.csite = s_csite;
      cl.env.site = a.site;
      cl.env.ncs = min(m, SC);
      cl.env.ci = ci;
      cl.env.si = a.site[scand[ci]];
      cl.env.site_i = scand[ci];
      a.pref[first + ci].word = 0;
      int r = clip_piece(cl, m);
      n64 += cl.n64;
      nex += cl.nex;
      if (r == CLIP_FULL) {  // out of vertex slots: the global variant redoes the piece with the same candidates
        if (LDS) push_overflow(a, make_int4(di.x, t, first + ci, first));
        else atomicOr(a.status, ST_SLOW_CAPACITY);
        continue;
      }
      if (r == CLIP_OK) {
        n_pairs += (unsigned long long)(long long)sd.sign;
        emit_alone(cl, sd, t, first + ci, a);
      }
    }
    __syncthreads();  // the candidate list is rewritten by the next item
  }
  for (int off = 32; off > 0; off >>= 1) {
    n_pairs += __shfl_xor(n_pairs, off);
    n64 += __shfl_xor(n64, off);
    nex += __shfl_xor(nex, off);
  }
  if (lane == 0) {
    if (n_pairs) stat_add(a, C_PAIRS, n_pairs);
    if (n64) stat_add(a, C_FP64, n64);
    if (nex) stat_add(a, C_EXACT, nex);
  }
}

// ---------------------------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------------------------
// The piece count is known on the device only: a grid of several times the wavefronts that fit the chip takes the
// chunks in grid-stride order (workgroups past the last chunk exit at once).
template <typename T, int SLOTS>
static hipError_t launch_pieces(const ShapeArgs& a, hipStream_t s) {
  const int grid = std::max(1, std::min(a.pcap / CHUNK, 8192));
  hipLaunchKernelGGL((k_clip_pieces<T, SLOTS>), dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_candidates(const ShapeArgs& a, hipStream_t s) {
  if (a.nitems == 0) return hipSuccess;
  hipLaunchKernelGGL(k_candidates, dim3(a.nitems), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_clip_pieces(const ShapeArgs& a, int precision, int slots, hipStream_t s) {
  if (a.nitems == 0) return hipSuccess;
  if (precision == RPD_FP64) return launch_pieces<double, 16>(a, s);
  if (slots == 12) return launch_pieces<float, 12>(a, s);
  return launch_pieces<float, 16>(a, s);
}

size_t slow_scratch_bytes(int waves) { return (size_t)waves * SlowScratch::bytes; }

// the first SLOW_LDS_ITEMS items by the LDS variant, the rest by the global one (whose waves exit at once when there
// is no rest); the item count is read on the device
hipError_t launch_clip_slow(const ShapeArgs& a, unsigned char* scratch, int waves, hipStream_t s) {
  const int lds_waves = waves < SLOW_LDS_ITEMS ? waves : SLOW_LDS_ITEMS;
  hipLaunchKernelGGL(k_clip_slow<true>, dim3(lds_waves), dim3(64), 0, s, a, scratch, 0, SLOW_LDS_ITEMS);
  hipLaunchKernelGGL(k_clip_slow<false>, dim3(waves), dim3(64), 0, s, a, scratch, SLOW_LDS_ITEMS, INT_MAX);
  return hipGetLastError();
}

}  // namespace rpd
